"""Every launch of a call fits a dispatch (at most 2^32 - 1 work-items), or the
call says UNSUPPORTED with nothing launched. A host program stands in for HIP's
launch call, which records the grids: sizes that no test could hold in memory
are checked on the CPU, with pointers that nothing reads."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_2509_23866_amd")

PROGRAM = r"""
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include "dart.h"

static long long launches, largest;

/* found before the ones of HIP's library: the program is searched first */
static dim3 grid_, block_;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
    grid_ = grid, block_ = block;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared,
                                                hipStream_t* stream) {
    *grid = grid_, *block = block_, *shared = 0, *stream = 0;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t,
                                      hipStream_t) {
    const long long items = (long long)grid.x * grid.y * grid.z * block.x * block.y * block.z;
    ++launches;
    if (items > largest) largest = items;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

int main(int, char** v) {
    const long long T = atoll(v[1]), d = atoll(v[2]), V = atoll(v[3]), rows = atoll(v[4]),
                    cols = atoll(v[5]);
    const unsigned flags = (unsigned)atoi(v[6]);
    void* const p = (void*)4096;
    const dart_status_t st = dart_lmhead_backward_ex(
        p, T, d, d, p, V, d, (const int32_t*)p, (const float*)p, (const float*)p, (const float*)p,
        1.f, p, d, p, d, rows, cols, flags, p, (size_t)1 << 60, (hipStream_t)0);
    printf("%d %lld %lld\n", (int)st, launches, largest);
    return 0;
}
"""


@pytest.fixture(scope="module")
def backward(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("launches")
    (d / "p.cpp").write_text(PROGRAM)
    exe = str(d / "p")
    subprocess.run([cxx, "-O1", "-D__HIP_PLATFORM_AMD__=1", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), str(d / "p.cpp"), "-o", exe, "-rdynamic",
                    "-L", LIBDIR, "-ldart", f"-Wl,-rpath,{LIBDIR}"], check=True)

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True)
        return tuple(map(int, out.stdout.split()))

    return run


@pytest.mark.parametrize("flags", [1, 1 | 4])
@pytest.mark.parametrize("T,d,V,cols", [
    (4096, 3584, 32000, 32000),
    (1 << 22, 4096, 16, 8),    # T d = 2^34: rows skipped, their sums put back over all of dhidden
    (4800000, 3584, 32000, 16000),
    (4800000, 3584, 32000, 32000),
    (0x7FFFFFFF, 8, 16, 8),
])
def test_backward_launches_fit_a_dispatch(backward, T, d, V, cols, flags):
    """At any T d: what is scattered back over [T, d] is launched in a bounded grid."""
    status, launches, largest = backward(T, d, V, 1 << 16, cols, flags)
    assert status == 0 and launches > 0
    assert largest <= 0xFFFFFFFF
