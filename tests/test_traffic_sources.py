"""The stencil's traffic record lapses with every source its kernels and their
launch rules are built from: each local header that dslash.hip includes,
directly or through another, is in the record's list."""
import os
import re

from paper_1010_2592_amd import rocprof_summary as rs

CSRC = "paper_1010_2592_amd/csrc"


def included(name, seen):
    if name in seen or not os.path.exists(os.path.join(rs.ROOT, CSRC, name)):
        return seen
    seen.add(name)
    with open(os.path.join(rs.ROOT, CSRC, name)) as f:
        for inc in re.findall(r'^#include "([^"]+)"', f.read(), re.M):
            included(inc, seen)
    return seen


def test_every_source_of_the_stencil_is_listed():
    need = {f"{CSRC}/{n}" for n in included("dslash.hip", set())} | {f"{CSRC}/solver.hip"}
    assert need <= set(rs.STENCIL_SOURCES)
