"""The one-launch scalar stages run on the CPU, a block at a time and wavefront
by wavefront (tests/emu): however a stage ends -- its gate closed, a breakdown
of alpha or beta, the Krylov space exhausted, an MR step cut short -- no two
wavefronts touch a word without a barrier between them where one writes it,
all of them wait at the same barriers, and the state does not depend on which
wavefront runs ahead.  Built with g++ from the library's sources; the accesses
are the ones the compiler's thread-sanitizer calls report."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1010_2592_amd", "csrc")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("stages")
    exe = str(d / "check")
    inc = ["-I", os.path.join(HERE, "emu"), "-I", CSRC, "-I", HERE]
    common = [gxx, "-O1", "-std=c++17", "-w", *inc, "-c"]
    subprocess.run([*common, "-fsanitize=thread", os.path.join(HERE, "scalar_stage_check.cpp"), "-o", str(d / "s.o")],
                   check=True)
    subprocess.run([*common, os.path.join(HERE, "emu", "block_emu.cpp"), "-o", str(d / "e.o")], check=True)
    subprocess.run([gxx, str(d / "s.o"), str(d / "e.o"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode in (0, 1), r.stderr
    return r.stdout.splitlines()


def test_no_races_and_common_barriers(lines):
    bad = [x for x in lines if " ok run" not in x]
    assert not bad, "\n".join(bad)


@pytest.mark.parametrize("what,end", [("alpha breaks down", "on 0 broken 1"), ("beta breaks down", "on 0 broken 1"),
                                      ("beta, exhausted", "on 0 broken 0 exhausted 1")])
def test_the_runs_reach_their_ends(lines, what, end):
    assert any(x.startswith(what) and end in x for x in lines)
