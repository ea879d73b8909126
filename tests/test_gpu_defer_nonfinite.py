"""A breakdown whose Mv output is not finite (a_scale so large that S u_0
overflows): no step completes, so the deferred single pass has nothing to add
to the zero solutions.  It must not read the output, whose
coefficient is zero (0 x inf): y, the solutions and the reported residuals are
those of the per-step form."""
import numpy as np
import pytest

import workloads as wl
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu
DIMS = (4, 4, 4, 8)


@pytest.mark.parametrize("form", ["basis", "explicit"])
@pytest.mark.parametrize("l", [1, 2, 4])
def test_overflow_in_the_first_step(l, form):
    from paper_1010_2592_amd import msb
    ctx = msb.Context(msb.Lattice(DIMS, -2.0, 0.05, -1), cuda(wl.gauge_links(DIMS, 0.6, 3)))
    b = cuda(1e10 * wl.gaussian_source(DIMS, 4, 2))
    sig, w = np.array([0.5, 1.0, 2.0]), np.array([1.0, 0.5, 0.25])
    kw = dict(want_shifts=True, allow=(msb.BREAKDOWN,))
    y0, i0, x0 = ctx.mshift_bicgstabl(b, 1e305, sig, w, l, 1e-8, 50, 1, **kw)
    y1, i1, x1 = ctx.mshift_bicgstabl(b, 1e305, sig, w, l, 1e-8, 50, 1, flags=msb.DEFERRED | (msb.SEED_BASIS if form == "basis" else 0),
                                      **kw)
    assert not host(y0).any() and not host(x0).any()
    assert not host(y1).any() and not host(x1).any()
    assert np.isfinite(i0.shift_resid).all() and np.array_equal(i0.shift_resid, i1.shift_resid)
    assert np.array_equal(i0.shift_iters, i1.shift_iters)
    ctx.close()
