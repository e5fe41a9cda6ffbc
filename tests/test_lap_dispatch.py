"""The Laplacian's launches, on the host alone: laplace.hip compiled without its device side, the
HIP runtime's launch calls replaced by a recorder.  Past the sizes where the chip is not full
anyway, a launch without sums leaves at most a fifth of its lanes without a site, however small
the slices are."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cxxabi.h>
#include <cstdlib>
#include "laplace.hip"

static std::map<const void *, std::string> names;
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
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t)
{
    printf("%u|%u|%s\n", g.x, b.x, names[f].c_str());
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}
thread_local laph_ctx *g_current_ctx;
void laph_fail(int code, const char *, ...) { throw LaphError{code}; }

int main(int argc, char **argv)
{
    for (int k = 1; k + 1 < argc; k += 2) {
        laph_ctx c;
        c.g.ns = atoi(argv[k]);
        c.g.nt = atoi(argv[k + 1]);
        c.g.V3 = (long)c.g.ns * c.g.ns * c.g.ns;
        c.g.V = c.g.V3 * c.g.nt;
        double2 v[1];
        double sums[1];
        for (int with = 0; with < 2; with++) {
            printf("%d|%d|%d|%d|", c.g.ns, c.g.nt, with, lap_blocks(c.g));
            lap_fused(&c, v, v, 0, nullptr, 0, v, 0, 1.0, 0.0, 0.0, v, 0, with ? sums : nullptr);
        }
    }
}
"""

LATTICES = [(2, 2), (2, 8), (4, 8), (8, 16), (12, 24), (14, 16), (14, 20), (16, 10), (16, 12), (16, 32), (24, 16), (24, 128),
            (12, 28), (14, 18), (16, 14), (2, 2048), (2, 8192), (4, 640), (4, 1024), (6, 160), (6, 256), (10, 60)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("needs the HIP compiler")
    tmp = tmp_path_factory.mktemp("lap")
    src, obj, exe = (str(tmp / n) for n in ("p.hip", "p.o", "p"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-O0", "-std=c++17", "-fPIE", "--offload-host-only", "-I",
                    os.path.join(ROOT, "paper_1104_3870_amd", "csrc"), "-c", src, "-o", obj],
                   check=True, capture_output=True, timeout=300)
    # (the device code image the host side refers to is not there, and never read)
    subprocess.run(["g++", obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"], check=True, capture_output=True,
                   timeout=100)
    out = subprocess.run([exe] + [str(n) for l in LATTICES for n in l], check=True, capture_output=True, text=True,
                         timeout=100).stdout
    res = {}
    for line in filter(None, out.split("\n")):
        ns, nt, with_sums, blocks, grid, lanes, kernel = line.split("|")
        res[int(ns), int(nt), int(with_sums)] = (int(blocks), int(grid), int(lanes), kernel)
    assert len(res) == 2 * len(LATTICES)
    return res


def test_lanes_have_sites(launches):
    for ns, nt in LATTICES:
        _, grid, lanes, kernel = launches[ns, nt, 0]
        per_site = 3 if "k_lap_rows" in kernel else 1
        V = ns ** 3 * nt
        assert grid * lanes >= per_site * V
        if V > 49152:
            assert grid * lanes < 1.25 * per_site * V + lanes, (ns, nt, kernel, grid)


def test_sums_per_slice(launches):
    """A workgroup's sums belong to one slice: lap_blocks of them each."""
    for ns, nt in LATTICES:
        blocks, grid, lanes, kernel = launches[ns, nt, 1]
        assert grid == blocks * nt and "<true" in kernel
        assert blocks * lanes >= (3 if "k_lap_rows" in kernel else 1) * ns ** 3


def test_lanes_per_site(launches):
    """Three lanes a site up to 768 workgroups of 64 sites, where they were measured the faster."""
    for ns, nt in LATTICES:
        _, _, _, kernel = launches[ns, nt, 0]
        assert ("k_lap_rows" in kernel) == (-(-ns ** 3 // 64) * nt <= 768), (ns, nt, kernel)
