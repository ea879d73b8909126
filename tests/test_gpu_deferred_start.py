"""The deferred single pass starts its shift vectors by writing them: a source
that never iterates (zero) must still get zero solutions, also where the
library's own buffers hold those of an earlier call, and a batch with one must
leave its other members as they are alone (the same bits: every right-hand
side's sums and updates run in its own rows)."""
import numpy as np
import pytest

import workloads as wl
from oracle import pfe
from tests.helpers import A_SCALE_BOUND, cuda, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["explicit", "basis", "mixed"])
@pytest.mark.parametrize("want", [False, True])
def test_zero_source_among_others(form, want):
    from paper_1010_2592_amd import msb
    dims = (4, 4, 4, 8)
    flags = msb.DEFERRED | {"explicit": 0, "basis": msb.SEED_BASIS, "mixed": msb.MIXED}[form]
    ctx = msb.Context(msb.Lattice(dims, -2.0, 0.05, -1), cuda(wl.gauge_links(dims, 0.6, 3)))
    b = wl.gaussian_source(dims, 4, 3)
    sig, w = pfe.neuberger(7)

    def solve(x):
        y, info, xs = ctx.mshift_bicgstabl(cuda(x), A_SCALE_BOUND, sig, w, 2, 1e-8, 500, 1, flags=flags, want_shifts=want)
        return host(y), info, None if xs is None else host(xs)
    full = solve(b)                      # fills the library's buffers
    z = b.copy()
    z[1] = 0.0
    y, info, xs = solve(z)
    assert not y[1].any() and not info.shift_iters[1].any()
    for r in (0, 2):
        assert np.array_equal(y[r], full[0][r])
    if want:
        assert not xs[1].any()
        assert np.array_equal(xs[[0, 2]], full[2][[0, 2]])
    ctx.close()
