"""The stencil's two forms and the chunked form's groups of right-hand sides at
the edges of their rules: one lane per site with a block per chunk and group,
or four wavefronts per chunk and right-hand side.  Every form adds a site's
hops in one order, so a batch is bitwise the single right-hand sides; and the
oracle at 1e-14 (the operator sums about 70 products per component; FP64
rounding stays some units below 1e-15 of the output's norm)."""
import numpy as np
import pytest

import workloads as wl
from oracle import dirac as od
from tests.helpers import cuda, rel
from tests.test_gpu_wilson import oracle_apply

pytestmark = pytest.mark.gpu


# (lattice, right-hand sides): less than one chunk; partial last chunk; batches
# on either side of the split form's limits (1024 and, for 2 and 3 right-hand
# sides, 1536 blocks); groups of 1 to 4 (one right-hand side per wavefront) and
# Lx = 16, whose x-neighbours come from the lanes
@pytest.mark.parametrize("dims,nrhs", [((3, 2, 2, 2), 2), ((5, 3, 2, 7), 7), ((8, 8, 8, 8), 15), ((8, 8, 8, 8), 16),
                                       ((8, 8, 8, 8), 17), ((16, 8, 8, 31), 2), ((16, 8, 8, 32), 3), ((12, 10, 9, 30), 3),
                                       ((9, 7, 11, 24), 5), ((16, 4, 6, 40), 13)])
@pytest.mark.parametrize("flags", [0, 1 | 2, 4])
def test_forms_match_single_rhs(dims, nrhs, flags):
    from paper_1010_2592_amd import msb
    U = wl.gauge_links(dims, 0.6, 3 + sum(dims))
    op = od.Dirac(U, dims, -2.0, 0.11, -1)
    v = wl.gaussian_source(dims, 9, nrhs)
    ctx = msb.Context(msb.Lattice(dims, -2.0, 0.11, -1), cuda(U))
    x = cuda(v)
    for extra in (0, msb.MIXED):
        batch = ctx.wilson_apply(x, flags | extra).cpu().numpy()
        for r in range(nrhs):
            assert np.array_equal(batch[r], ctx.wilson_apply(x[r:r + 1], flags | extra)[0].cpu().numpy()), (extra, r)
        if not extra:
            some = [0, nrhs - 1]
            assert rel(batch[some], oracle_apply(op, v[some], flags)) <= 1e-14
    ctx.close()


def test_one_group_of_a_large_lattice_matches_single_rhs():
    """2048 chunks: one block per chunk takes all right-hand sides in turn."""
    from paper_1010_2592_amd import msb
    import torch
    dims, nrhs = (16, 16, 16, 32), 6
    ctx = msb.Context(msb.Lattice(dims, -2.0, 0.05, -1), cuda(wl.gauge_links(dims, 0.5, 1003)))
    x = cuda(wl.gaussian_source(dims, 5, nrhs))
    batch = ctx.wilson_apply(x, 1)
    for r in range(nrhs):
        assert torch.equal(batch[r], ctx.wilson_apply(x[r:r + 1], 1)[0])
    ctx.close()


@pytest.mark.parametrize("dims,nrhs", [((5, 3, 2, 7), 1), ((8, 8, 8, 8), 15), ((8, 8, 8, 8), 18), ((16, 8, 8, 32), 3)])
@pytest.mark.parametrize("pass_", [1, 2])
def test_solve_of_a_batch_is_that_of_its_members(dims, nrhs, pass_):
    """The epilogues (inner products, y of the double pass): forced iterations,
    a batch against each member alone, whose reductions run in the same order."""
    from paper_1010_2592_amd import msb
    ctx = msb.Context(msb.Lattice(dims, -2.0, 0.05, -1), cuda(wl.gauge_links(dims, 0.6, 12)))
    x = cuda(wl.gaussian_source(dims, 9, nrhs))
    sig, w = msb.neuberger_pfe(4)
    kw = dict(force_iters=np.array([2, 2, 1, 1]))
    y = ctx.mshift_bicgstabl(x, 0.02, sig, w, 2, 1e-8, 100, pass_, **kw)[0].cpu().numpy()
    assert np.isfinite(y.view(np.float64)).all()
    for r in (0, nrhs - 1):
        one = ctx.mshift_bicgstabl(x[r:r + 1], 0.02, sig, w, 2, 1e-8, 100, pass_, **kw)[0].cpu().numpy()[0]
        assert np.array_equal(y[r], one), r
    ctx.close()
