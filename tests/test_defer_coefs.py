"""The deferred single pass's coefficients for l = 1..8 and up to 64 shifts
(64 x 19 items in a block of 512), iterations cut short after any step, a shift
whose recurrences stop: the device code on the CPU (tests/emu) against the
per-step recurrences in long double.  Bound, in units of eps times the same
recurrences on absolute values: a coefficient passes through at most l steps
and the MR step, each at most 2 l + 6 complex operations deep, of at most
4 eps each."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1010_2592_amd", "csrc")


@pytest.fixture(scope="module")
def worst(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("defer") / "check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-w", "-I", os.path.join(HERE, "emu"), "-I", CSRC, "-I", HERE,
                    os.path.join(HERE, "defer_coef_check.cpp"), os.path.join(HERE, "emu", "block_emu.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=200).stdout
    return {int(a): float(b) for a, b in (x.split() for x in out.splitlines())}


@pytest.mark.parametrize("l", range(1, 9))
def test_coefficients(worst, l):
    assert worst[l] <= 4 * (l + 1) * (2 * l + 6)
