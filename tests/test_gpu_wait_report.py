"""A wait inside a sweep that is given up (forced by a bound of one poll; the
launch itself ends) is reported by the next call, and by a call that
synchronizes; a context with the default bound is not affected."""
import numpy as np
import pytest

import pd_inputs as P
from gpu_util import dev, gpu_context

pytestmark = pytest.mark.gpu


def _context():
    sc = P.scene_small(16, 15, 12, h=1.0, region_top_layers=2, seed=5)
    c = gpu_context(sc, interior="levels")
    x = dev(sc.rest)
    import torch
    return c, x, torch.ones_like(x), torch.zeros(3 * c.m, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("sweep", ["condense", "backsub"])
def test_given_up_wait_is_reported(sweep):
    import torch
    from paper_2008_01541_amd._lib import PDError
    c, x, f, y2 = _context()
    c.condense_rhs(f, y2)
    torch.cuda.synchronize()
    c.set_wait_limit(1)
    if sweep == "condense":
        c.condense_rhs(f, y2)
    else:
        c.backsub(torch.ones_like(y2), x)
    torch.cuda.synchronize()
    with pytest.raises(PDError):
        c.region_gather(x, y2)
    with pytest.raises(PDError):
        c.condense_rhs(f, y2)
    c.close()


def test_synchronizing_call_reports_it():
    from paper_2008_01541_amd._lib import PDError
    c, x, f, y2 = _context()
    c.set_wait_limit(1)
    c.condense_rhs(f, y2)
    with pytest.raises(PDError):
        c.displacement_change(x, x.clone())
    c.close()


def test_default_bound_and_bad_bounds():
    from paper_2008_01541_amd._lib import PDError
    c, x, f, y2 = _context()
    with pytest.raises(PDError):
        c.set_wait_limit(0)
    c.condense_rhs(f, y2)
    c.backsub(y2, x)
    assert np.isfinite(c.displacement_change(x, x.clone())).all()
    c.close()
