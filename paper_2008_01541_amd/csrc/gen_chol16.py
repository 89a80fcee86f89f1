"""Writes chol16_steps.inc: the elimination of a 16 x 16 diagonal block (and
of 64 further rows that ride along) as one scheduled inline-asm block, for
tile_factor_f64.h (run from this directory; the output is committed).

Lane r of every row of 16 lanes holds row r of the block in a[]; x[] holds one
more row per lane, solved against the factor on the way.  Pivot C:
  d     = a[C] of lane C (DPP row_newbcast),
  y     = 1/sqrt(d): the estimate y0 (v_rsq_f64, relative error up to about
          5e-8) and one third-order step, u = d y0, e = 1 - u y0,
          y = y0 + (y0 e) (1/2 + 3 e / 8),
  a[C] *= y, x[C] *= y,
  a[S] -= L(S, C) a[C] and x[S] -= L(S, C) x[C] for S = C+1 .. 15, with
          L(S, C) = a[C] of lane S broadcast by the DPP operand of v_fmac_f64.
The next pivot needs a[C+1] only, so its broadcast and square root run in the
issue slots between the updates that are left over from step C: a list
scheduler orders the instructions by the length of the path that hangs on
each (an FP64 instruction issues in 4 cycles and its result can be used after
8; v_rsq_f64 takes 16 and 20).  Two orders are kept by the scheduler because
the hardware does not interlock them: a DPP read of a VGPR comes at least two
instructions after the VALU write of it, and the use of a v_rsq_f64 result at
least one instruction after it.  s_nop fills what no instruction can.
"""

DPP = "row_mask:0xf bank_mask:0xf"
N = 16


class Ins:
    __slots__ = ("text", "dst", "src", "dpp", "rsq", "succ", "npred", "ready", "after", "prio", "pos")

    def __init__(self, text, dst, src, dpp=None, rsq=False):
        self.text, self.dst, self.src, self.dpp, self.rsq = text, dst, src, dpp, rsq


def program():
    ins = []
    add = lambda *a, **k: ins.append(Ins(*a, **k))  # noqa: E731
    for c in range(N):
        # d is kept apart by parity: the next pivot's may be broadcast early
        d, ac, xc = f"d{c % 2}", f"a{c}", f"x{c}"
        add(f"v_mov_b64_dpp %[{d}], %[{ac}] row_newbcast:{c} {DPP}", d, [ac], dpp=ac)
        add(f"v_rsq_f64 %[y0], %[{d}]", "y0", [d], rsq=True)
        add(f"v_mul_f64 %[u], %[{d}], %[y0]", "u", [d, "y0"])
        add("v_fma_f64 %[e], -%[u], %[y0], 1.0", "e", ["u", "y0"])
        add("v_fma_f64 %[g], %[e], %[k375], 0.5", "g", ["e"])
        add("v_mul_f64 %[e], %[y0], %[e]", "e", ["y0", "e"])
        add("v_fma_f64 %[y], %[e], %[g], %[y0]", "y", ["e", "g", "y0"])
        add(f"v_mul_f64 %[{ac}], %[{ac}], %[y]", ac, [ac, "y"])
        add(f"v_mul_f64 %[{xc}], %[{xc}], %[y]", xc, [xc, "y"])
        for s in range(c + 1, N):
            add(f"v_fmac_f64_dpp %[a{s}], -%[{ac}], %[{ac}] row_newbcast:{s} {DPP}", f"a{s}",
                [f"a{s}", ac], dpp=ac)
            add(f"v_fmac_f64_dpp %[x{s}], -%[{ac}], %[{xc}] row_newbcast:{s} {DPP}", f"x{s}",
                [f"x{s}", ac, xc], dpp=ac)
    return ins


def schedule(ins):
    """Order of the instructions ("s_nop k" where a wait state is left empty)
    and the modelled cycles."""
    n = len(ins)
    preds = [[] for _ in range(n)]          # (index, kind): raw, war, waw
    writer, readers = {}, {}
    for i, p in enumerate(ins):
        for r in p.src:
            if r in writer:
                preds[i].append((writer[r], "dpp" if p.dpp == r else "raw"))
        for j in readers.get(p.dst, []):
            preds[i].append((j, "war"))
        if p.dst in writer:
            preds[i].append((writer[p.dst], "waw"))
        for r in p.src:
            readers.setdefault(r, []).append(i)
        writer[p.dst] = i
        readers[p.dst] = []
    lat = lambda j, kind: 0 if kind == "war" else (20 if ins[j].rsq else 8)  # noqa: E731
    succ = [[] for _ in range(n)]
    for i in range(n):
        for j, kind in preds[i]:
            succ[j].append((i, kind))
    path = [0] * n
    for i in range(n - 1, -1, -1):
        path[i] = max([lat(i, k) + (4 if k == "dpp" else 0) + path[s] for s, k in succ[i]],
                      default=4)
    done, pos, order, t = {}, {}, [], 0
    left = [len(p) for p in preds]
    avail = [i for i in range(n) if left[i] == 0]
    while avail:
        best, when = None, None
        for i in avail:
            at = t
            for j, kind in preds[i]:
                at = max(at, done[j] + lat(j, kind))
                if kind == "dpp":            # two instructions between
                    at = max(at, t + 4 * max(0, pos[j] + 3 - len(order)))
                elif kind == "raw" and ins[j].rsq:
                    at = max(at, t + 4 * max(0, pos[j] + 2 - len(order)))
            key = (max(at, t), -path[i], i)
            if best is None or key < best:
                best, when = key, i
        i = when
        need = 0
        for j, kind in preds[i]:
            if kind == "dpp":
                need = max(need, pos[j] + 3 - len(order))
            elif kind == "raw" and ins[j].rsq:
                need = max(need, pos[j] + 2 - len(order))
        for _ in range(need):
            order.append(None)
        t = max(best[0], t)
        done[i], pos[i] = t, len(order)
        order.append(i)
        t += 16 if ins[i].rsq else 4
        avail.remove(i)
        for s, _ in succ[i]:
            left[s] -= 1
            if left[s] == 0:
                avail.append(s)
    return order, t


def check(ins, order):
    """The order computes what the program does, and keeps the two distances."""
    at = {i: k for k, i in enumerate(order) if i is not None}
    assert sorted(at) == list(range(len(ins)))
    writer, readers = {}, {}
    for i, p in enumerate(ins):
        for r in p.src:
            if r in writer:
                j = writer[r]
                gap = 3 if p.dpp == r else (2 if ins[j].rsq else 1)
                assert at[i] - at[j] >= gap
            readers.setdefault(r, []).append(i)
        for j in readers.get(p.dst, []):
            assert at[i] >= at[j]
        if p.dst in writer:
            assert at[i] > at[writer[p.dst]]
        writer[p.dst] = i
        readers[p.dst] = []


def main():
    ins = program()
    order, cycles = schedule(ins)
    check(ins, order)
    lines = ["s_nop 1"]                      # a[0] may have just been written
    for i in order:
        lines.append("s_nop 0" if i is None else ins[i].text)
    body = "\n".join(f'      "{x}\\n\\t"' for x in lines)
    outs = ", ".join([f'[a{i}] "+v"(a[{i}])' for i in range(N)] +
                     [f'[x{i}] "+v"(x[{i}])' for i in range(N)] +
                     [f'[{r}] "=&v"({r})' for r in ("d0", "d1", "y0", "u", "e", "g", "y")])
    out = ["// Generated by gen_chol16.py; do not edit.  Elimination of a 16 x 16 block, one",
           "// row per lane of every 16 lanes in a[], and of one more row per lane in x[]; returns",
           "// the last pivot, which is not a number if any pivot was not positive.  "
           f"Modelled: {cycles} cycles.",
           "__device__ __forceinline__ double chol16_eliminate(double (&a)[16], double (&x)[16]) {",
           "  double d0, d1, y0, u, e, g, y;",
           "  const double k375 = 0.375;",
           "  asm volatile(", body,
           f"      : {outs}", '      : [k375] "v"(k375));', "  return d1;", "}"]
    open("chol16_steps.inc", "w").write("\n".join(out) + "\n")
    print(len(order), "instructions,", sum(o is None for o in order), "empty,", cycles, "cycles")


if __name__ == "__main__":
    main()
