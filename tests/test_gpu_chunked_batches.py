"""The chunked stencil's epilogues at the sizes where it can go wrong, with
batches that the library's own rule sends there (asserted on the host): a
partial last chunk, whole chunks per time slice (chunks walked t fastest) and
not, Lx = 16 with its x-neighbours from the lanes of a row, with a whole z-t
plane per wavefront (16 x 4) and with wavefronts that straddle planes (16 x 3),
groups of right-hand sides and one group for all of them, FP64 and FP32.  Every
form adds a site's hops in one order and a chunk's sums too, so a batch is
bitwise each of its members alone, which take the split form."""
import numpy as np
import pytest

import workloads as wl
from oracle import cg as ocg
from oracle import dirac as od
from oracle import pfe
from tests.helpers import A_SCALE_BOUND, cuda, host, rel
from tests.stencil_rule import MV, MV_Y, MVV, PLAIN, SV, rule
from tests.test_gpu_wilson import oracle_apply

pytestmark = pytest.mark.gpu


def context(dims, mu=0.05):
    from paper_1010_2592_amd import msb
    return msb.Context(msb.Lattice(dims, -2.0, mu, -1), cuda(wl.gauge_links(dims, 0.6, 11 + sum(dims))))


# 50400 sites: 788 chunks, the last half full, and one group for all
@pytest.mark.parametrize("dims,nrhs,groups", [((3, 5, 2, 90), 24, 6), ((6, 4, 10, 30), 10, 3), ((8, 8, 8, 8), 18, 5),
                                              ((16, 4, 2, 64), 9, 3), ((16, 3, 3, 75), 8, 2), ((16, 3, 3, 350), 5, 1)])
@pytest.mark.parametrize("flags", [0, 1 | 2, 4])
def test_operator(dims, nrhs, groups, flags):
    from paper_1010_2592_amd import msb
    for fp64 in (True, False):
        form, n, _ = rule(dims, nrhs, PLAIN, g5=flags == 4, fp64=fp64)
        assert form == "chunk" and n in (groups, 1)
    mu = 0.11
    op = od.Dirac(wl.gauge_links(dims, 0.6, 11 + sum(dims)), dims, -2.0, mu, -1)
    v = wl.gaussian_source(dims, 9, nrhs)
    ctx = context(dims, mu)
    x = cuda(v)
    for extra in (0, msb.MIXED):
        batch = host(ctx.wilson_apply(x, flags | extra))
        for r in range(nrhs):
            assert np.array_equal(batch[r], host(ctx.wilson_apply(x[r:r + 1], flags | extra))[0]), (extra, r)
        if not extra:
            some = [0, nrhs - 1]
            assert rel(batch[some], oracle_apply(op, v[some], flags)) <= 1e-14
    ctx.close()


# pass 1: Mv with r~ and without (the last one); pass 2: with y; a point
# source's r~ is a list, its Mv the epilogue without r~; mixed: FP32, and FP64
# in the reliable updates
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 66), ((16, 3, 3, 75), 26), ((5, 3, 4, 64), 72)])
@pytest.mark.parametrize("source", ["gauss", "point"])
@pytest.mark.parametrize("pass_,mixed", [(1, False), (2, False), (1, True), (2, True)])
def test_solves(dims, nrhs, source, pass_, mixed):
    from paper_1010_2592_amd import msb
    for fp64 in ((True, False) if mixed else (True,)):
        for epi in (PLAIN, MV, MV_Y, SV):
            assert rule(dims, nrhs, epi, fp64=fp64)[0] == "chunk"
    ctx = context(dims)
    b = wl.gaussian_source(dims, 9, nrhs)
    if source == "point":
        b = np.zeros_like(b)
        for r in range(nrhs):
            b[r, r % 12, 5 * r] = 1.0 + 0.5j
    x = cuda(b)
    sig, w = pfe.neuberger(3)
    kw = dict(flags=msb.MIXED if mixed else 0, force_iters=np.array([2, 2, 1]), allow=(msb.OK, msb.REDUCED_ACCURACY))
    y = host(ctx.mshift_bicgstabl(x, A_SCALE_BOUND, sig, w, 2, 1e-8, 100, pass_, **kw)[0])
    assert np.isfinite(y.view(np.float64)).all() and y.any(axis=(1, 2)).all()
    for r in (0, 3, nrhs // 2, nrhs - 1):
        one = host(ctx.mshift_bicgstabl(x[r:r + 1], A_SCALE_BOUND, sig, w, 2, 1e-8, 100, pass_, **kw)[0])[0]
        assert np.array_equal(y[r], one), r
    ctx.close()


# CG's epilogue, Re <v, out> from the operand it adds; FP64 against the oracle
# at the bound of the CG tests
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 16), ((16, 3, 3, 75), 7), ((5, 3, 4, 64), 18)])
@pytest.mark.parametrize("pass_", [1, 2, 3])
def test_cg(dims, nrhs, pass_):
    assert rule(dims, nrhs, MVV)[0] == "chunk" and rule(dims, nrhs, PLAIN)[0] == "chunk"
    ctx = context(dims, 0.0)
    op = od.Dirac(wl.gauge_links(dims, 0.6, 11 + sum(dims)), dims, -2.0, 0.0, -1)
    b = wl.gaussian_source(dims, 6, nrhs)
    x = cuda(b)
    sig, w = pfe.neuberger(4)
    force = np.array([8, 6, 3, 1])
    y, info, _ = ctx.mshift_cg(x, A_SCALE_BOUND, sig, w, 1e-10, 100, pass_, force_iters=force)
    y = host(y)
    for r in (0, nrhs // 2, nrhs - 1):
        one, i1, _ = ctx.mshift_cg(x[r:r + 1], A_SCALE_BOUND, sig, w, 1e-10, 100, pass_, force_iters=force)
        assert np.array_equal(y[r], host(one)[0]), r
        assert np.array_equal(info.shift_resid[r], i1.shift_resid[0])
    want = ocg.mshift_cg(lambda v: op.a_op(v, A_SCALE_BOUND), b[nrhs - 1], sig, w, 1e-10, 100, 1, force_iters=force)[0]
    assert rel(y[nrhs - 1], want) <= 1e-10
    ctx.close()
