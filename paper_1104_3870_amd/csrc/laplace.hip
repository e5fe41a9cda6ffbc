// Gauge-covariant 3D Laplacian (Sec. II) and its Chebyshev transform (Sec. IV), batched
// over all time slices.  The fused kernel computes
//     out = alpha * (Lap in) + beta * in + gamma * prev
// which is one step of T_k = 2 B T_{k-1} - T_{k-2}, B = 1 + c (Lap + lambda_C).
#include "laplace.h"

namespace {

constexpr int kLapLanes = 256;

// the three sums of a block of W waves to sums[b][3]
template <int W>
__device__ __forceinline__ void lap_sums(double dre, double dim, double nrm, unsigned b, double *__restrict__ sums)
{
    __shared__ double red[3][W];
    for (int w = 32; w > 0; w >>= 1) {
        dre += __shfl_down(dre, w, 64);
        dim += __shfl_down(dim, w, 64);
        nrm += __shfl_down(nrm, w, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = dre;
        red[1][threadIdx.x >> 6] = dim;
        red[2][threadIdx.x >> 6] = nrm;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int w = 0; w < W; w++) v += red[threadIdx.x][w];
        sums[(long)b * 3 + threadIdx.x] = v;
    }
}

// one lane per (slice t, spatial site), a workgroup's sites in one slice, or (FLAT) in several;
// vectors of slice t start at base + t * stride.  DOT: block sums of <dot, out> and |out|^2 (see
// lap_fused)
template <bool DOT, bool FLAT>
__global__ __launch_bounds__(kLapLanes) void k_lap(const double2 *__restrict__ us, const double2 *__restrict__ in,
                                             long in_stride, const double2 *__restrict__ prev, long prev_stride,
                                             double2 *__restrict__ out, long out_stride, int ns, int nt, long V,
                                             double alpha, double beta, double gamma, int nblk,
                                             const double2 *__restrict__ dot, long dot_stride, double *__restrict__ sums)
{
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    const long V3 = V / nt;
    // (32-bit division: 27 links of 16 bytes a site keep V far below 2^32)
    const unsigned flat = b * kLapLanes + threadIdx.x;
    const int t = (int)(FLAT ? flat / (unsigned)V3 : b / nblk);
    const long r = FLAT ? (long)flat - (long)t * V3 : (long)(b - (unsigned)t * nblk) * kLapLanes + threadIdx.x;
    const long s = (long)t * V3 + r;
    double dre = 0.0, dim = 0.0, nrm = 0.0;
    if (FLAT ? s < V : r < V3) {
    int x = (int)(r % ns);
    long q = r / ns;
    int y = (int)(q % ns);
    int z = (int)(q / ns);
    const double2 *vin = in + t * in_stride;
    double2 acc[3];
    double2 self[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        self[a] = vin[r * 3 + a];
        acc[a] = cscale(self[a], -6.0);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) {
        int xp = x, yp = y, zp = z, xm = x, ym = y, zm = z;
        if (k == 0) {
            xp = x + 1 == ns ? 0 : x + 1;
            xm = x == 0 ? ns - 1 : x - 1;
        } else if (k == 1) {
            yp = y + 1 == ns ? 0 : y + 1;
            ym = y == 0 ? ns - 1 : y - 1;
        } else {
            zp = z + 1 == ns ? 0 : z + 1;
            zm = z == 0 ? ns - 1 : z - 1;
        }
        long rp = xp + (long)ns * (yp + (long)ns * zp);
        long rm = xm + (long)ns * (ym + (long)ns * zm);
        long sm = rm + (long)t * V3;
        double2 vp[3], vm[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            vp[a] = vin[rp * 3 + a];
            vm[a] = vin[rm * 3 + a];
        }
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int c = 0; c < 3; c++) {
                acc[a] = cadd(acc[a], cmul(us[(long)(k * 9 + a * 3 + c) * V + s], vp[c]));
                acc[a] = cadd(acc[a], cconjmul(us[(long)(k * 9 + c * 3 + a) * V + sm], vm[c]));
            }
    }
    double2 *vo = out + t * out_stride;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        double2 o = cadd(cscale(acc[a], alpha), cscale(self[a], beta));
        if (prev) o = cadd(o, cscale(prev[t * prev_stride + r * 3 + a], gamma));
        vo[r * 3 + a] = o;
        if (DOT) {
            const double2 q = dot[t * dot_stride + r * 3 + a];
            dre += q.x * o.x + q.y * o.y;
            dim += q.x * o.y - q.y * o.x;
            nrm += cnorm2(o);
        }
    }
    }
    if (DOT) lap_sums<kLapLanes / 64>(dre, dim, nrm, b, sums);
}

// The same with one lane per (slice, site, colour row), three waves for a workgroup's 64 sites
// of one slice: on small lattices the kernel above leaves most of the chip idle while each of
// its few waves waits for 72 loads
template <bool DOT>
__global__ __launch_bounds__(192) void k_lap_rows(const double2 *__restrict__ us, const double2 *__restrict__ in,
                                             long in_stride, const double2 *__restrict__ prev, long prev_stride,
                                             double2 *__restrict__ out, long out_stride, int ns, int nt, long V,
                                             double alpha, double beta, double gamma, int nblk,
                                             const double2 *__restrict__ dot, long dot_stride, double *__restrict__ sums)
{
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    const int t = (int)(b / nblk);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), row = wave;
    const unsigned V3 = (unsigned)(V / nt), r = (b - (unsigned)t * nblk) * 64 + (threadIdx.x & 63);
    double dre = 0.0, dim = 0.0, nrm = 0.0;
    if (r < V3) {
    const unsigned q1 = r / (unsigned)ns, q2 = q1 / (unsigned)ns;
    const int x = (int)(r - q1 * ns), y = (int)(q1 - q2 * ns), z = (int)q2;
    const double2 *vin = in + t * in_stride;
    const double2 self = vin[r * 3 + row];
    double2 acc = cscale(self, -6.0);
    us += (long)t * V3;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        int xp = x, yp = y, zp = z, xm = x, ym = y, zm = z;
        if (k == 0) {
            xp = x + 1 == ns ? 0 : x + 1;
            xm = x == 0 ? ns - 1 : x - 1;
        } else if (k == 1) {
            yp = y + 1 == ns ? 0 : y + 1;
            ym = y == 0 ? ns - 1 : y - 1;
        } else {
            zp = z + 1 == ns ? 0 : z + 1;
            zm = z == 0 ? ns - 1 : z - 1;
        }
        const unsigned rp = xp + ns * (yp + ns * zp), rm = xm + ns * (ym + ns * zm);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            acc = cadd(acc, cmul(us[(long)(k * 9 + row * 3 + c) * V + r], vin[rp * 3 + c]));
            acc = cadd(acc, cconjmul(us[(long)(k * 9 + c * 3 + row) * V + rm], vin[rm * 3 + c]));
        }
    }
    double2 o = cadd(cscale(acc, alpha), cscale(self, beta));
    if (prev) o = cadd(o, cscale(prev[t * prev_stride + r * 3 + row], gamma));
    out[t * out_stride + r * 3 + row] = o;
    if (DOT) {
        const double2 q = dot[t * dot_stride + r * 3 + row];
        dre = q.x * o.x + q.y * o.y;
        dim = q.x * o.y - q.y * o.x;
        nrm = cnorm2(o);
    }
    }
    if (DOT) lap_sums<3>(dre, dim, nrm, b, sums);
}

}  // namespace

// workgroups of 64 sites up to which three lanes a site are faster: three for each of the 256 CUs,
// which hold them all at once (a step, one lane / three: 4^3 x 8 5.1 / 3.2 us, 8^3 x 16 5.5 / 3.3;
// 648 workgroups, 12^3 x 24, 5.7 / 5.4; 756, 12^3 x 28, 6.2 / 5.8; 768, 16^3 x 12, 6.1 / 5.7 and
// 8^3 x 96 5.8 / 5.5; 774, 14^3 x 18, 6.4 / 6.9; 896, 16^3 x 14, 6.4 / 7.1; 24^3 x 128 249 / 315)
constexpr long kLapRowsMost = 768;
// slices that leave half of a one-lane workgroup idle or more (2^3, 4^3): several of them share one
// (a step of 2^3 x 8192 6.5 us, a slice each 89; 4^3 x 1024 6.5, 12.8; but 6^3 x 256 6.3, 6.0, 10^3 x
// 48 6.5, 5.9), and where sums per slice are asked for, the workgroups of 64 sites take them (29 us
// and 6.6)
static bool lap_small_slice(const Geom &g) { return 2 * g.V3 <= kLapLanes; }
static int lap_slice_blocks(const Geom &g, bool rows)
{
    const int sites = rows ? 64 : kLapLanes;
    return (int)((g.V3 + sites - 1) / sites);
}
static bool lap_rows(const Geom &g, bool sums)
{
    return (long)lap_slice_blocks(g, true) * g.nt <= kLapRowsMost || (sums && lap_small_slice(g));
}

int lap_blocks(const Geom &g) { return lap_slice_blocks(g, lap_rows(g, true)); }

void lap_fused(laph_ctx *c, const double2 *us, const double2 *in, long in_stride, const double2 *prev,
               long prev_stride, double2 *out, long out_stride, double alpha, double beta, double gamma,
               const double2 *dot, long dot_stride, double *sums)
{
    const bool rows = lap_rows(c->g, sums), flat = !rows && lap_small_slice(c->g);
    const int nblk = lap_slice_blocks(c->g, rows);
    const dim3 grid(flat ? nblocks_for(c->g.V, kLapLanes) : (unsigned)(nblk * (long)c->g.nt));
    auto launch = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, grid, dim3(lanes), 0, c->stream, us, in, in_stride, prev, prev_stride, out,
                           out_stride, c->g.ns, c->g.nt, c->g.V, alpha, beta, gamma, nblk, dot, dot_stride, sums);
    };
    if (rows)
        sums ? launch(k_lap_rows<true>, 192) : launch(k_lap_rows<false>, 192);
    else if (flat)
        launch(k_lap<false, true>, kLapLanes);
    else
        sums ? launch(k_lap<true, false>, kLapLanes) : launch(k_lap<false, false>, kLapLanes);
    LAPH_HIP(hipGetLastError());
}

// out = T_order(B) in, B = 1 + cc (Lap + lamC); w0, w1 scratch of the same shape
void cheb_apply(laph_ctx *c, const double2 *us, const double2 *in, long in_stride, double2 *out, long out_stride,
                double2 *w0, double2 *w1, long w_stride, double lamL, double lamC, int order, double *sums)
{
    double cc = 2.0 / (lamL - lamC);
    double b0 = 1.0 + cc * lamC;  // B = cc * Lap + b0
    if (order == 0) {
        lap_fused(c, us, in, in_stride, nullptr, 0, out, out_stride, 0.0, 1.0, 0.0, in, in_stride, sums);
        return;
    }
    if (order == 1) {
        lap_fused(c, us, in, in_stride, nullptr, 0, out, out_stride, cc, b0, 0.0, in, in_stride, sums);
        return;
    }
    // T_1 -> w0; then T_k = 2 B T_{k-1} - T_{k-2}, rotating buffers so T_order lands in out
    const double2 *tm2 = in;
    long s2 = in_stride;
    double2 *bufs[2] = {w0, w1};
    lap_fused(c, us, in, in_stride, nullptr, 0, w0, w_stride, cc, b0, 0.0);
    const double2 *tm1 = w0;
    long s1 = w_stride;
    int nb = 1;
    for (int k = 2; k <= order; k++) {
        double2 *dst;
        long sd;
        if (k == order) {
            dst = out;
            sd = out_stride;
        } else {
            dst = bufs[nb];
            sd = w_stride;
            nb ^= 1;
        }
        lap_fused(c, us, tm1, s1, tm2, s2, dst, sd, 2.0 * cc, 2.0 * b0, -1.0, in, in_stride,
                  k == order ? sums : nullptr);
        tm2 = tm1;
        s2 = s1;
        tm1 = dst;
        s1 = sd;
    }
}

static double2 *prepare_soa(laph_ctx *c, const double *U)
{
    double2 *us = (double2 *)ctx_named(c, "lap.us", (size_t)27 * c->g.V * 16);
    smeared_links_to_soa(c, U, us);
    return us;
}

extern "C" int laph_laplacian_apply(laph_ctx_t c, const double *U, const double *v, double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(U && v && out && v != out, LAPH_EINVAL, "bad arguments");
    double2 *us = prepare_soa(c, U);
    long V3 = c->g.V3;
    // one launch covers all slices: a "slice stride" of V3*3 makes the layout contiguous
    lap_fused(c, us, (const double2 *)v, V3 * 3, nullptr, 0, (double2 *)out, V3 * 3, 1.0, 0.0, 0.0);
    LAPH_API_END(c)
}

extern "C" int laph_chebyshev_apply(laph_ctx_t c, const double *U, double lamL, double lamC, int order,
                                    const double *v, double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(U && v && out && v != out && order >= 0 && lamL > lamC, LAPH_EINVAL, "bad arguments");
    double2 *us = prepare_soa(c, U);
    long V3 = c->g.V3;
    size_t bytes = (size_t)c->g.V * 3 * 16;
    double2 *w0 = (double2 *)ctx_named(c, "cheb.w0", bytes), *w1 = (double2 *)ctx_named(c, "cheb.w1", bytes);
    cheb_apply(c, us, (const double2 *)v, V3 * 3, (double2 *)out, V3 * 3, w0, w1, V3 * 3, lamL, lamC, order, nullptr);
    LAPH_API_END(c)
}
