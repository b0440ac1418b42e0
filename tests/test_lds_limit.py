"""The LDS limit of a kernel is raised on each device that launches it, and a refusal is tried again
(CPU: a program with its own hipFuncSetAttribute and hipLaunchKernel before the runtime's)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2602_14016_amd")

DRIVER = r"""
#include <cstdio>
#include "%s"

static int asked = 0;
static bool refuse = false;
static hipError_t last = hipSuccess;
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
    ++asked;
    return refuse ? last = hipErrorInvalidValue : hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

int main() {
    pa::cd field[1];
    pa::Dims d{};
    d.N = 1024;
    d.B = 1;
    d.K = 341;
    d.KX = 342;
    d.KXP = 344;
    d.KY = 683;
    d.tpb = d.atpb = 4;
    d.cus = 256;
    d.lds_max = 163840;
    pa::RowArgs a{};
    for (auto& p : a.yin) p = field;
    for (auto& p : a.yout) p = field;
    a.tw = field;
    const struct { int device; bool refuse; } runs[] = {{0, true}, {0, false}, {0, false}, {1, true}, {1, false},
                                                        {1, false}, {0, false}, {70, false}, {70, false}};
    for (const auto& r : runs) {
        d.device = (short)r.device;
        refuse = r.refuse;
        const hipError_t e = pa::launch_row_sq(d, a, nullptr);
        std::printf("%%d %%d %%d\n", (int)e, asked, (int)hipGetLastError());
    }
    return 0;
}
"""


@pytest.mark.timeout(600)
def test_limit_is_raised_per_device_and_retried(tmp_path):
    from paper_2602_14016_amd.build import ARCH, BUILD_DIR, COMMON, DEVICE_FLAGS, HIPCC, build
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    if not os.path.exists(os.path.join(BUILD_DIR, "kern_1024.o")):
        build(verbose=False)
    objects = [os.path.join(BUILD_DIR, f) for f in sorted(os.listdir(BUILD_DIR))
               if f.endswith(".o") and f.startswith("kern")]
    src, obj, exe = tmp_path / "driver.hip", tmp_path / "driver.o", tmp_path / "driver"
    src.write_text(DRIVER % os.path.join(PKG, "csrc", "kernels.hpp"))
    subprocess.run([HIPCC] + COMMON + DEVICE_FLAGS + ["-c", str(src), "-o", str(obj)], check=True)
    subprocess.run([HIPCC, f"--offload-arch={ARCH}", str(obj)] + objects + ["-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=120, check=True).stdout
    rows = [tuple(map(int, l.split())) for l in out.splitlines()]
    # (result, limits asked for so far, error left): refused, raised, kept; the second device the
    # same; the first still kept; devices past the 64th ask each time
    assert rows == [(1, 1, 0), (0, 2, 0), (0, 2, 0), (1, 3, 0), (0, 4, 0), (0, 4, 0), (0, 4, 0), (0, 5, 0), (0, 6, 0)]
