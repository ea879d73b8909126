"""The stencil's choice of form and groups against the launch times behind it
(us per launch, measured on gfx950): no launch may go to a form that took 4 %
longer than the other, nor may a batch be cut into groups where that did."""
import shutil

import pytest

from tests.stencil_rule import MV, MV_Y, PLAIN, SV, rule

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")

D = {"8^4": (8, 8, 8, 8), "12^4": (12, 12, 12, 12), "8^3x32": (8, 8, 8, 32), "10x9x7x14": (10, 9, 7, 14),
     "12^3x24": (12, 12, 12, 24), "16^3x12": (16, 16, 16, 12), "16^4": (16, 16, 16, 16), "16^3x24": (16, 16, 16, 24),
     "16^3x32": (16, 16, 16, 32)}
# lattice, right-hand sides, epilogue, gamma5 on the input, FP64: split, one group, groups of four
TIMES = [
    ("8^4", 12, MV, 0, 1, 13.4, 30.0, 15.7), ("8^4", 16, PLAIN, 0, 1, 13.9, 25.4, 11.8),
    ("8^4", 32, MV, 0, 1, 31.5, 69.6, 28.6), ("8^3x32", 4, SV, 0, 1, 14.5, 13.6, 13.7),
    ("8^3x32", 12, MV, 0, 1, 41.5, 40.0, 39.0), ("8^3x32", 24, PLAIN, 1, 1, 57.8, 42.3, 53.0),
    ("10x9x7x14", 6, SV, 0, 1, 14.7, 19.0, 17.2), ("10x9x7x14", 12, PLAIN, 1, 1, 21.2, 23.5, 20.5),
    ("12^4", 6, MV, 0, 1, 31.8, 36.4, 36.5), ("12^4", 12, MV_Y, 0, 1, 60.5, 77.2, 80.1),
    ("12^3x24", 2, PLAIN, 0, 1, 17.4, 18.5, 18.7), ("12^3x24", 3, SV, 0, 1, 24.8, 27.0, 27.2),
    ("12^3x24", 3, MV_Y, 0, 1, 29.6, 40.8, 41.0), ("12^3x24", 3, MV_Y, 0, 0, 21.6, 27.3, 27.3),
    ("12^3x24", 3, PLAIN, 1, 1, 22.4, 26.6, 26.6), ("12^3x24", 24, MV, 0, 1, 266.2, 197.7, 182.0),
    ("12^3x24", 12, PLAIN, 1, 1, 91.4, 70.7, 79.6), ("16^3x12", 2, MV_Y, 0, 1, 27.9, 38.8, 38.8),
    ("16^3x12", 2, PLAIN, 1, 1, 22.5, 29.7, 29.7), ("16^3x12", 5, MV_Y, 0, 1, 60.4, 77.4, 79.4),
    ("16^3x12", 24, PLAIN, 1, 1, 274.7, 170.6, 211.6), ("16^4", 2, MV_Y, 0, 1, 31.7, 41.2, 41.3),
    ("16^4", 12, PLAIN, 0, 1, 154.2, 101.1, 105.1), ("16^4", 12, MV, 0, 1, 210.1, 134.7, 143.0),
    ("16^4", 24, PLAIN, 1, 1, 329.6, 199.8, 237.5), ("16^3x24", 2, PLAIN, 0, 1, 41.1, 34.6, 34.4),
    ("16^3x24", 2, MV, 0, 1, 44.6, 46.5, 46.7), ("16^3x24", 2, MV_Y, 0, 0, 31.0, 40.9, 41.0),
    ("16^3x24", 3, PLAIN, 1, 1, 47.0, 52.3, 52.6), ("16^3x32", 2, MV, 0, 1, 68.2, 61.9, 62.4),
    ("16^3x32", 2, MV_Y, 0, 1, 75.0, 81.5, 81.2), ("16^3x32", 3, PLAIN, 1, 1, 78.8, 71.0, 71.5),
]


@pytest.mark.parametrize("case", TIMES, ids=lambda c: f"{c[0]}-{c[1]}-epi{c[2]}{'-g5' if c[3] else ''}{'' if c[4] else '-fp32'}")
def test_no_launch_goes_to_a_slower_form(case):
    name, nrhs, epi, g5, fp64, split, one, groups = case
    form, n, _ = rule(D[name], nrhs, epi, bool(g5), bool(fp64))
    took = split if form == "split" else one if n == 1 else groups
    assert took <= 1.04 * min(split, one, groups), (form, n)


@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 8), 1), ((24, 24, 24, 48), 1), ((3, 2, 2, 2), 5), ((16, 3, 3, 75), 9),
                                       ((8, 8, 8, 8), 17), ((16, 16, 16, 32), 12)])
@pytest.mark.parametrize("epi", [PLAIN, MV, MV_Y])
def test_the_grid_covers_every_chunk_and_group(dims, nrhs, epi):
    V = dims[0] * dims[1] * dims[2] * dims[3]
    nch = -(-V // 64)
    for fp64 in (False, True):
        form, groups, blocks = rule(dims, nrhs, epi, fp64=fp64)
        assert 1 <= groups <= nrhs and (nrhs > 1 or form == "split")
        assert blocks % 8 == 0 and blocks >= nch * groups
