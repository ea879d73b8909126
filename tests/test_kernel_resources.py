"""Registers of kernels whose speed rests on the wavefronts a SIMD holds, as
the compiler reports them for gfx950 with the library's own flags: one register
too many halves the wavefronts in flight and shows in no result."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1010_2592_amd import build as lib

SOURCE = """
#include "stencil_dev.h"
using namespace msb;
using namespace msb::dev;
template <typename T, int EPI, bool G5IN>
__global__ __launch_bounds__(64 * CHUNK_WAVES) void chunk(DslashArgs<T> a) {
    dslash_chunk<T, EPI, G5IN, CHUNK_WAVES>(a, blockIdx.x);
}
template __global__ void chunk<double, EPI_MV, false>(DslashArgs<double>);
template __global__ void chunk<double, EPI_MVN, false>(DslashArgs<double>);
template __global__ void chunk<double, EPI_MV_Y, false>(DslashArgs<double>);
"""


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("res")
    src = d / "kernels.hip"
    src.write_text(SOURCE)
    r = subprocess.run([lib._hipcc(), *lib.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        str(src), "-o", str(d / "kernels.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"(Function Name|VGPRs|AGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): *(\S+)", line)
        if m and m.group(1) == "Function Name":
            name = subprocess.run(["c++filt", m.group(2)], capture_output=True, text=True).stdout.split("(")[0].strip()
            out[name] = {}
        elif m and name:
            out[name][m.group(1).split()[0]] = int(m.group(2))
    return out


# FP64 chunked stencil: two blocks per CU by the links they stage, so two
# wavefronts per SIMD
@pytest.mark.parametrize("epi", [1, 5, 2])
def test_chunked_stencil_keeps_two_wavefronts(report, epi):
    k = report[f"void chunk<double, {epi}, false>"]
    assert k["Occupancy"] >= 2 and k["AGPRs"] == 0 and k["ScratchSize"] == 0, k
