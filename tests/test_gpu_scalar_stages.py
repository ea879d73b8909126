"""The one-launch scalar stages (sixteen wavefronts summing the partials side
by side) at the ends of their ranges, against the persistent launch, whose
scalar stages sum the same partials in a 256-wide block: the same order, so
the same bits.  And the deferred update's coefficients (one work-item per
shift and basis index) with more items than its block, against the per-step
single pass."""
import numpy as np
import pytest

import workloads as wl
from oracle import pfe
from tests.helpers import A_SCALE_BOUND, cuda, host, problem, rel
from tests.test_gpu_solver import ctx_for, oracle_run, parity_bound

pytestmark = pytest.mark.gpu


def context(dims):
    from paper_1010_2592_amd import msb
    return msb.Context(msb.Lattice(dims, -2.0, 0.05, -1), cuda(wl.gauge_links(dims, 0.5, 17)))


# fewer partials than a wavefront; more than the 4096 of one round of loads
# (4224 chunks); 64 shifts, one per lane; l = 6, 27 pairs of the Gram matrix
@pytest.mark.parametrize("dims,l,ns", [((4, 4, 4, 2), 1, 1), ((5, 3, 4, 7), 2, 64), ((8, 8, 8, 8), 6, 33),
                                       ((16, 16, 16, 66), 3, 5)])
def test_sums_are_the_persistent_launch_s(dims, l, ns):
    from paper_1010_2592_amd import msb
    ctx = context(dims)
    b = cuda(wl.gaussian_source(dims, 7, 1))
    sig, w = pfe.neuberger(ns)
    kw = dict(force_iters=np.minimum(2, 1 + np.arange(ns) % 2), want_shifts=True)
    y0, i0, x0 = ctx.mshift_bicgstabl(b, A_SCALE_BOUND, sig, w, l, 1e-8, 50, 1, **kw)
    y1, i1, x1 = ctx.mshift_bicgstabl(b, A_SCALE_BOUND, sig, w, l, 1e-8, 50, 1, flags=msb.PERSISTENT, **kw)
    assert np.array_equal(host(y0), host(y1)) and np.array_equal(host(x0), host(x1))
    assert np.array_equal(i0.shift_iters, i1.shift_iters) and np.array_equal(i0.shift_resid, i1.shift_resid)
    ctx.close()


# 46 shifts: 46 x 19 items in a block of 512; the two forms of the update agree
# to rounding (1e-11 as in the deferred form's own tests)
@pytest.mark.parametrize("l,ns", [(1, 3), (4, 46)])
def test_deferred_coefficients_match_per_step(l, ns):
    from paper_1010_2592_amd import msb
    dims = (4, 4, 4, 8)
    ctx = context(dims)
    b = cuda(wl.gaussian_source(dims, 8, 2))
    sig, w = pfe.neuberger(ns)
    kw = dict(force_iters=1 + np.arange(ns) % 3, want_shifts=True)
    y0, i0, x0 = ctx.mshift_bicgstabl(b, A_SCALE_BOUND, sig, w, l, 1e-8, 50, 1, **kw)
    for flags in (msb.DEFERRED, msb.DEFERRED | msb.SEED_BASIS):
        y1, i1, x1 = ctx.mshift_bicgstabl(b, A_SCALE_BOUND, sig, w, l, 1e-8, 50, 1, flags=flags, **kw)
        assert np.array_equal(i0.shift_iters, i1.shift_iters)
        assert rel(host(y1), host(y0)) <= 1e-11
        assert max(rel(host(x1)[r, s], host(x0)[r, s]) for r in range(2) for s in range(ns)) <= 1e-11
    ctx.close()


# the Gram matrix's sums, halved over a wavefront: 12 to 72 values, the last
# in two parts (90 values: the basis form's test at l = 8)
@pytest.mark.parametrize("l", [2, 3, 5, 7])
def test_gram_sums_match_oracle(l):
    from paper_1010_2592_amd import msb
    wk, U, op, a, sg, w, b = problem("4x4x4x8")
    force = np.full(len(sg), 2)
    want = oracle_run(op, a, b[0], sg, w, l, wk.tol, 2, 1, force=force)[0]
    bound = parity_bound(op, a, b[0], sg, w, l, wk.tol, force, want)
    ctx = ctx_for(wk, U)
    y, _, _ = ctx.mshift_bicgstabl(cuda(b), a, sg, w, l, wk.tol, 2, 1, force_iters=force,
                                   allow=(msb.OK, msb.NOT_CONVERGED))
    assert rel(host(y)[0], want) <= bound
    ctx.close()
