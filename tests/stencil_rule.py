"""The stencil's form and groups for a launch, from the library's header
(tests/stencil_rule.cpp, built with g++): what the tests of the forms ask to
know that a batch takes the form they are about."""
import functools
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1010_2592_amd", "csrc")
PLAIN, MV, MV_Y, SV, MVV = 0, 1, 2, 3, 4


@functools.lru_cache(maxsize=1)
def _program():
    d = tempfile.mkdtemp(prefix="stencil_rule")
    exe = os.path.join(d, "rule")
    subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-w", "-I", os.path.join(HERE, "emu"), "-I", CSRC,
                    os.path.join(HERE, "stencil_rule.cpp"), "-o", exe], check=True)
    return exe


def rules(calls):
    """[(form, groups, blocks)] of calls (dims, nrhs, epi, gamma5 on the input, fp64)."""
    text = "".join("%d %d %d %d %d %d %d %d\n" % (epi, g5, fp64, *dims, nrhs) for dims, nrhs, epi, g5, fp64 in calls)
    out = subprocess.run([_program()], input=text, capture_output=True, text=True, check=True).stdout
    return [(f, int(g), int(n)) for f, g, n in (x.split() for x in out.splitlines())]


def rule(dims, nrhs, epi=PLAIN, g5=False, fp64=True):
    return rules([(dims, nrhs, epi, g5, fp64)])[0]
