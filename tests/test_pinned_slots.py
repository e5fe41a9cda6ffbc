"""The solver's pinned slots, on the host alone: solver.hip compiled without its device side, the
few runtime calls of the protocol replaced.  The memory has to be asked for as coherent (the host
reads it while the stream is busy), the numbers skip 0 and alternate between the two slots also
where they wrap, and a wait ends whatever the stream does: with the scalars once every right-hand
side carries the number, with an error where the stream failed or ended without them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "solver.hip"

static unsigned flags;
static int queries, answer_after;
static hipError_t answer;
static PinSlot *late;
static unsigned late_seq;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
hipError_t hipHostMalloc(void **p, size_t n, unsigned f)
{
    flags = f;
    *p = malloc(n);
    memset(*p, 0xff, n);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t)
{
    if (++queries < answer_after) return hipErrorNotReady;
    if (late)
        for (int r = 0; r < 3; r++) {
            late->s[r].iters = 100 + r;
            late->seq[r] = late_seq;
        }
    return answer;
}
const char *hipGetErrorString(hipError_t) { return ""; }
}
thread_local laph_ctx *g_current_ctx;
void laph_fail(int code, const char *, ...) { throw LaphError{code}; }

static int wait(laph_ctx *c, const Turn &t, std::vector<Scal> &h)
{
    try {
        wait_turn(c, t, 3, h);
    } catch (const LaphError &e) {
        return e.code;
    }
    return 0;
}

int main()
{
    laph_ctx c;
    Turn a = next_turn(&c), b = next_turn(&c);
    printf("coherent %d\n", (flags & hipHostMallocCoherent) != 0);
    printf("cleared %d\n", a.pin->seq[0] == 0 && b.pin->seq[31] == 0);
    printf("alternate %d\n", a.pin != b.pin && a.seq != b.seq);
    c.pin_seq = 0xfffffffeu;
    a = next_turn(&c);
    b = next_turn(&c);
    printf("wrap %d\n", a.seq == 0xffffffffu && b.seq != 0 && a.pin != b.pin && next_turn(&c).pin == a.pin);
    std::vector<Scal> h(3);
    // two of three right-hand sides there, the stream ends without the third
    b.pin->seq[0] = b.pin->seq[1] = b.seq;
    answer = hipSuccess;
    answer_after = 2;
    queries = 0;
    printf("ended %d %d\n", wait(&c, b, h), queries);
    answer = hipErrorLaunchFailure;
    queries = 0;
    printf("failed %d %d\n", wait(&c, b, h), queries);
    // the number arrives with the stream's end
    late = b.pin;
    late_seq = b.seq;
    answer = hipSuccess;
    queries = 0;
    printf("late %d %d %d\n", wait(&c, b, h), h[0].iters, h[2].iters);
    queries = 0;
    printf("there %d %d\n", wait(&c, b, h), queries);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the HIP compiler")
def test_slots(tmp_path):
    src, obj, exe = (str(tmp_path / n) for n in ("p.hip", "p.o", "p"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-O0", "-std=c++17", "-fPIE", "--offload-host-only", "-I",
                    os.path.join(ROOT, "paper_1104_3870_amd", "csrc"), "-c", src, "-o", obj],
                   check=True, capture_output=True, timeout=300)
    # (the device code image the host side refers to is not there, and never read)
    subprocess.run(["g++", obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"], check=True, capture_output=True,
                   timeout=100)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    got = dict(line.split(" ", 1) for line in out.strip().split("\n"))
    ehip = "5"
    assert got == {"coherent": "1", "cleared": "1", "alternate": "1", "wrap": "1", "ended": ehip + " 2",
                   "failed": ehip + " 2", "late": "0 100 102", "there": "0 0"}
