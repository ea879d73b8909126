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


def resources(src, out):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("hipcc not available")
    r = subprocess.run([lib._hipcc(), *lib.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        str(src), "-o", str(out / "kernels.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"(Function Name|VGPRs|AGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): *(\S+)", line)
        if m and m.group(1) == "Function Name":
            name = m.group(2)
            found[name] = {}
        elif m and name:
            found[name][m.group(1).split()[0]] = int(m.group(2))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True).stdout.splitlines()
    return {re.sub(r"msb::(\(anonymous namespace\)::)?", "", n).split("(")[0].strip(): v
            for n, v in zip(names, found.values())}


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    d = tmp_path_factory.mktemp("res")
    (d / "kernels.hip").write_text(SOURCE)
    return resources(d / "kernels.hip", d)


@pytest.fixture(scope="module")
def blas(tmp_path_factory):
    return resources(os.path.join(lib.CSRC, "blas.hip"), tmp_path_factory.mktemp("blas"))


# FP64 chunked stencil: two blocks per CU by the links they stage, so two
# wavefronts per SIMD
@pytest.mark.parametrize("epi", [1, 5, 2])
def test_chunked_stencil_keeps_two_wavefronts(report, epi):
    k = report[f"void chunk<double, {epi}, false>"]
    assert k["Occupancy"] >= 2 and k["AGPRs"] == 0 and k["ScratchSize"] == 0, k


@pytest.mark.parametrize("kernel,waves", [("k_r_update<float, 1, true, true, true>", 8),
                                          ("k_mr_update<float, 7, false, true>", 6),
                                          ("k_mr_update<float, 8, false, true>", 6)])
def test_vector_updates_keep_their_wavefronts(blas, kernel, waves):
    k = blas["void " + kernel]
    assert k["Occupancy"] >= waves and k["ScratchSize"] == 0, k
