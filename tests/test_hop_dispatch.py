"""Which kernel an FP64 hop launch takes, on the host alone: dslash.hip compiled without its
device side, the HIP runtime's launch calls replaced by a recorder.  Every epilogue mode has to
reach its own instantiation on every route (few pairs: the split kernel; 8, 16 or 32 right-hand
sides: staged, except the dot epilogue; else the rolled one), and a mode without one has to fail
instead of running another epilogue.  The bytes a launch reports to the timing are those of its
links, its clover term and every field it reads or writes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cxxabi.h>
#include <cstdlib>
#include <string>
#include "dslash.hip"

static std::map<const void *, std::string> names;
static std::string last;
static dim3 G, B;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, void *, void *,
                           int *)
{
    int st;
    char *d = abi::__cxa_demangle(dev, nullptr, nullptr, &st);
    names[host] = d ? d : dev;
    free(d);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { G = g; B = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *t)
{
    *g = G;
    *b = B;
    *s = 0;
    *t = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t) { last = names[f]; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}
thread_local laph_ctx *g_current_ctx;
void laph_fail(int code, const char *, ...) { throw LaphError{code}; }
static double bytes;
void timing_begin(laph_ctx *, hipEvent_t *a, hipEvent_t *b) { *a = *b = (hipEvent_t)1; }
void timing_end(laph_ctx *, hipEvent_t, hipEvent_t, double n, const char *) { bytes = n; }
const char *timing_label(const char *, const char *, int, int) { return ""; }

template <class F>
static void show(const char *what, int mode, long Vh, int R, F f)
{
    last = "none";
    try {
        f();
    } catch (const LaphError &e) {
        last = "error " + std::to_string(e.code);
    }
    printf("%s|%d|%ld|%d|%s\n", what, mode, Vh, R, last.c_str());
}

int main()
{
    laph_ctx c;
    for (int mode = 0; mode < 8; mode++) {
        for (long Vh : {256L, 1024L, 1025L, 32768L, 32769L, 65536L})
            for (int R : {1, 2, 8, 12, 16, 31, 32})
                show("launch", mode, Vh, R, [&] {
                    DslashArgs a{};
                    a.ns = 8;
                    a.nt = 4;
                    a.Vh = Vh;
                    a.R = R;
                    launch_dslash<S64, G64, C64>(&c, mode, a, nullptr);
                });
        show("staged", mode, 0, 32, [&] {
            launch_modes<S64, G64, C64, true>(mode, dim3(1), dim3(256), 0, nullptr, DslashArgs{});
        });
        show("split", mode, 0, 32, [&] { launch_split(mode, 64, nullptr, DslashArgs{}); });
    }
    // fields read beside the input: x, and y of the dot epilogue where it is another one
    const double f[2] = {};
    for (int mode : {M_PLAIN, M_INV_AFTER, M_INV_AFTER_DOT})
        for (int x = mode == M_INV_AFTER_DOT; x < 2; x++)
            for (int y = 0; y < (mode == M_INV_AFTER_DOT ? 2 : 1); y++) {
                DslashArgs a{};
                a.ns = 8;
                a.nt = 4;
                a.Vh = 1024;
                a.R = 4;
                a.x = x ? f : nullptr;
                a.dot_y = f + y;
                launch_dslash<S64, G64, C64>(&c, mode, a, nullptr);
                printf("bytes|%d|%d|%d|%.0f\n", mode, x, y, bytes);
            }
}
"""

PLAIN, INV, OF_SUM, CLOV_ADD, DOT = 0, 1, 2, 3, 6
EINVAL = "error 1"


def _want(what, mode, n, R):
    if mode not in (PLAIN, INV, OF_SUM, CLOV_ADD, DOT):
        return EINVAL
    if what == "split" or (what == "launch" and n <= 32768):
        return "k_dslash_split<%d>" % mode
    staged = what == "staged" or (R in (8, 16, 32) and mode != DOT)
    if staged and mode == DOT:
        return EINVAL
    return "k_dslash<S64, G64, C64, %d, true, %s>" % (mode, "true" if staged else "false")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the HIP compiler")
def test_every_mode_reaches_its_kernel(tmp_path):
    src, obj, exe = (str(tmp_path / n) for n in ("p.hip", "p.o", "p"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-O0", "-std=c++17", "-fPIE", "--offload-host-only", "-I",
                    os.path.join(ROOT, "paper_1104_3870_amd", "csrc"), "-c", src, "-o", obj],
                   check=True, capture_output=True, timeout=300)
    # (the device code image the host side refers to is not there, and never read)
    subprocess.run(["g++", obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"], check=True, capture_output=True,
                   timeout=100)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=100).stdout.split("\n")
    seen = 0
    for line in filter(None, out):
        what, mode, Vh, R, got = line.split("|")
        if what == "bytes":
            x, y = int(Vh), int(R)
            links, clover = 8 * 9 * 16, 0 if int(mode) == PLAIN else 72 * 8
            assert float(got) == 1024 * (links + clover + 4 * 12 * 16 * (2 + x + y)), line
            seen += 1
            continue
        assert _want(what, int(mode), int(Vh) * int(R), int(R)) in got, line
        seen += 1
    assert seen == 8 * (6 * 7 + 2) + 6
