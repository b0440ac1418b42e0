"""A context that cannot have a second stream recomputes in line and leaves no error behind (CPU).

api.hip's host code is compiled into a program whose own hipGetDevice, hipEventCreateWithFlags,
hipStreamCreateWithFlags and hipGetLastError stand before the runtime's: each creation is refused in
turn, and a refused call's error stays until it is asked for, as the runtime keeps it."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2602_14016_amd")

DRIVER = r"""
#include "%s"

static int refuse_at = 0, calls = 0;   // the call (1, 2, ...) that is refused
static hipError_t last = hipSuccess;
static hipError_t answer() {
    if (++calls != refuse_at) return hipSuccess;
    return last = hipErrorOutOfMemory;
}
extern "C" hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
extern "C" hipError_t hipGetDevice(int* d) { *d = 0; return answer(); }
extern "C" hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return answer(); }
extern "C" hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(0x10);
    return answer();
}

int main() {
    for (refuse_at = 1; refuse_at <= 5; ++refuse_at) {
        pa_ctx c{};
        c.d.N = 256;
        c.device = 0;
        c.prof_class = -1;
        calls = 0;
        (void)hipGetLastError();
        const bool beside = overlaps(&c, 50);
        const hipError_t left = hipGetLastError();
        std::printf("%%d %%d %%d %%d\n", refuse_at, (int)beside, (int)(c.side != nullptr), (int)left);
    }
    return 0;
}
"""


@pytest.mark.timeout(600)
def test_refused_second_stream_leaves_no_error(tmp_path):
    from paper_2602_14016_amd.build import ARCH, BUILD_DIR, COMMON, DEVICE_FLAGS, HIPCC, build
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    if not os.path.exists(os.path.join(BUILD_DIR, "misc.o")):
        build(verbose=False)
    objects = [os.path.join(BUILD_DIR, f) for f in sorted(os.listdir(BUILD_DIR)) if f.endswith(".o") and f != "api.o"]
    src, obj, exe = tmp_path / "driver.hip", tmp_path / "driver.o", tmp_path / "driver"
    src.write_text(DRIVER % os.path.join(PKG, "csrc", "api.hip"))
    flags = [f for f in COMMON if f != "-O3"] + ["-O1"]
    subprocess.run([HIPCC] + flags + DEVICE_FLAGS + ["-c", str(src), "-o", str(obj)], check=True)
    subprocess.run([HIPCC, f"--offload-arch={ARCH}", str(obj)] + objects + ["-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=120, check=True).stdout
    # refused at the device query, either event, the stream, and not at all
    assert [tuple(map(int, l.split())) for l in out.splitlines()] == [
        (1, 0, 0, 0), (2, 0, 0, 0), (3, 0, 0, 0), (4, 0, 0, 0), (5, 1, 1, 0)]
