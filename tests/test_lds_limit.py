"""The permission for more than 64 KB of dynamic LDS is asked for once per kernel and device.  Host only: the library's own header compiled
with two functions of the runtime in its place."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "free_internal.h"
static int device, asked[70], fail;
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
    if (fail) return hipErrorInvalidValue;
    ++asked[device];
    return hipSuccess;
}
namespace freemi { void note_hip_error(hipError_t) {} }
int main() {
    freemi::LdsLimit limit;
    for (int pass = 0; pass < 2; ++pass)
        for (int d : {0, 1, 63}) {
            device = d;
            if (!limit.allow(nullptr, 98304) || asked[d] != 1) return 1;
        }
    device = 2;
    fail = 1;
    if (limit.allow(nullptr, 98304)) return 2;                // refused: not remembered as allowed
    fail = 0;
    if (!limit.allow(nullptr, 98304) || asked[2] != 1) return 3;
    device = 65;                                              // beyond what is remembered: asked for every time
    if (!limit.allow(nullptr, 98304) || !limit.allow(nullptr, 98304) || asked[65] != 2) return 4;
    return 0;
}
"""


def test_once_per_device(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2511_20390_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=20).returncode == 0
