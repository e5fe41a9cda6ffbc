// Covariant displacements of colour fields and their momentum-projected overlaps (Sec. II:
// displacement types D^(j) of the quark lines D^(j) S Omega^-1 S D^(k)dag; Sec. III.B: the
// momentum projection of the meson function).
//
// A displaced, momentum-projected meson function of LapH-smeared fields D^(j) V_s a and
// D^(k) V_s b factorises through the overlaps O[t][n][m] = sum_x e^{-ip.x} (D^(j) v_n)^dag
// (D^(k) v_m) of displaced eigenvectors: M = e^{-ip.(d_j + d_k)/2} sum c_ab conj(a_an)
// O_nm b_bm, so the fields are displaced once per eigenvector, not once per quark line.
#include <cmath>

#include "laph_impl.h"
#include "zgemm_mfma.h"

namespace {

// out[t][j][x] = (D v_j)(x) for colour fields in the eigenvector layout [Nt][n][Ns^3][3]:
// one lane per site (t, x) forms the path's link product W(x) once (W = U(x) U(x+e) ...
// U(x+(len-1)e), or the product of the adjoints backwards) and applies it to v_j at the
// far end for every j, so each link is read once per site, not once per vector.  Bound by
// HBM.  A lane's result is 48 bytes, and storing it as three 16-byte pieces makes three
// partial writes of every cache line: a wave instead passes its 64 sites through LDS (its
// own 3 KB a vector, no barrier) and stores whole lines past the caches.  112 vectors on
// 24^3 x 128, three links: 3.75 ms (5.3 TB/s), with partial stores 4.6 ms; two or one vector
// in flight 3.77-3.8 ms.
constexpr int kDisLanes = 256, kDisVecs = 4;
typedef double vd2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(kDisLanes) void k_displace(const double2 *__restrict__ U, const double2 *__restrict__ v, double2 *__restrict__ out,
                           int ns, int nt, int n, int dir, int sign, int len)
{
    __shared__ double2 pass[kDisLanes / 64][kDisVecs][192];
    const long V3 = (long)ns * ns * ns, sites = (long)nt * V3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const long q0 = blockIdx.x * (long)kDisLanes + 64 * wave;  // the wave's first site
    if (q0 >= sites) return;
    // (lanes past the end work on the last site and store nothing)
    const long q = min(q0 + lane, sites - 1);
    const int t = (int)(q / V3);
    const long xyz = q - (long)t * V3;
    int c[3] = {(int)(xyz % ns), (int)((xyz / ns) % ns), (int)(xyz / ((long)ns * ns))};
    // W = product of the links from x to the far end, left to right
    double2 W[9];
#pragma unroll
    for (int e = 0; e < 9; e++) W[e] = make_double2((e % 4) == 0 ? 1.0 : 0.0, 0.0);
    int cur = c[dir];
    for (int k = 0; k < len; k++) {
        int s3[3] = {c[0], c[1], c[2]};
        const int nxt = ((cur + sign) % ns + ns) % ns;
        s3[dir] = sign > 0 ? cur : nxt;  // forward: U_d(cur); backward: U_d(cur - e)^dag
        const long site = s3[0] + (long)ns * (s3[1] + (long)ns * s3[2]) + V3 * t;
        const double2 *L = U + (site * 4 + dir) * 9;
        double2 Lm[9], R[9];
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                const double2 u = sign > 0 ? L[a * 3 + b] : L[b * 3 + a];
                Lm[a * 3 + b] = sign > 0 ? u : make_double2(u.x, -u.y);
            }
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                double2 acc = make_double2(0.0, 0.0);
#pragma unroll
                for (int m = 0; m < 3; m++) acc = cadd(acc, cmul(W[a * 3 + m], Lm[m * 3 + b]));
                R[a * 3 + b] = acc;
            }
#pragma unroll
        for (int e = 0; e < 9; e++) W[e] = R[e];
        cur = nxt;
    }
    int f[3] = {c[0], c[1], c[2]};
    f[dir] = cur;
    const long far = f[0] + (long)ns * (f[1] + (long)ns * f[2]);
    // the lane's three elements of the wave's 192 contiguous ones (site e / 3, colour e % 3)
    long to[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int e = lane + 64 * k;
        const long s = q0 + e / 3, ts = s / V3;
        to[k] = s < sites ? (ts * n * V3 + (s - ts * V3)) * 3 + e % 3 : -1;
    }
    const double2 *vf = v + ((long)t * n * V3 + far) * 3;
    // kDisVecs vectors' loads in flight per lane
    for (int j0 = 0; j0 < n; j0 += kDisVecs) {
        double2 w[kDisVecs][3];
#pragma unroll
        for (int u = 0; u < kDisVecs; u++)
#pragma unroll
            for (int a = 0; a < 3; a++) w[u][a] = vf[(long)min(j0 + u, n - 1) * V3 * 3 + a];
#pragma unroll
        for (int u = 0; u < kDisVecs; u++) {
            double2 *row = pass[wave][u];
#pragma unroll
            for (int a = 0; a < 3; a++)
                row[3 * lane + a] = cadd(cadd(cmul(W[a * 3], w[u][0]), cmul(W[a * 3 + 1], w[u][1])),
                                         cmul(W[a * 3 + 2], w[u][2]));
        }
        // the wave's lanes read each other's values (LDS keeps a wave's order; this keeps the compiler's)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int u = 0; u < kDisVecs; u++) {
            if (j0 + u >= n) break;
            double2 *o = out + (long)(j0 + u) * V3 * 3;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const double2 r = pass[wave][u][lane + 64 * k];
                if (to[k] >= 0) __builtin_nontemporal_store(vd2{r.x, r.y}, (vd2 *)&o[to[k]]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// phase[x] = exp(-2 pi i k.x / Ns) on one slice
__global__ void k_phase(double2 *ph, int ns, int k0, int k1, int k2)
{
    const long V3 = (long)ns * ns * ns;
    const long x = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (x >= V3) return;
    const int cx = (int)(x % ns), cy = (int)((x / ns) % ns), cz = (int)(x / ((long)ns * ns));
    // the integer phase index reduced mod Ns keeps the argument small and exact
    const long m = (((long)k0 * cx + (long)k1 * cy + (long)k2 * cz) % ns + ns) % ns;
    double s, c;
    sincospi(-2.0 * (double)m / ns, &s, &c);
    ph[x] = make_double2(c, s);
}

// O[t][n][m] = sum_{x, c} conj(a[t][n][x][c]) ph[x] b[t][m][x][c]: per slice the product
// A^dag (ph B) over K = 3 Ns^3 on the FP64 matrix cores, the conjugate and the phase applied
// while staging; with parts > 1 the sum over x in that many pieces, out[t][piece][n][m]
struct OverlapS {
    const double2 *pa, *pb, *ph;
    double2 *out;
    int M, N, K;  // na, nb, 3 Ns^3 / parts
    int tiles_m, tiles_n;
    long batches;  // nt parts
    int parts;
    __device__ zg::Side side(const double2 *p, long bt, int rows, int conj, const double2 *phase) const
    {
        const long t = bt / parts, q = bt - t * parts, full = (long)K * parts;
        return {p + t * rows * full + q * K, full, 1, rows, conj, phase ? phase + q * (K / 3) : nullptr};
    }
    __device__ zg::Side a(long bt) const { return side(pa, bt, M, 1, nullptr); }
    __device__ zg::Side b(long bt) const { return side(pb, bt, N, 0, ph); }
    __device__ void store(long bt, int m, int n, double re, double im) const
    {
        out[(bt * M + m) * (long)N + n] = make_double2(re, im);
    }
};

// out[j][t][beta][p] = sum_m O[t][p][m] b[j][t][beta][m]; one lane per output element
__global__ void k_overlap_apply(const double2 *__restrict__ O, int na, int nb, const double2 *__restrict__ b,
                                long nrt, double2 *__restrict__ out, int nt)
{
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (q >= nrt * 4 * na) return;
    const int p = (int)(q % na);
    const long rb = q / na;  // (j, t, beta)
    const int t = (int)((rb / 4) % nt);
    const double2 *orow = O + ((long)t * na + p) * nb;
    const double2 *bv = b + rb * nb;
    double2 acc = make_double2(0.0, 0.0);
    for (int m = 0; m < nb; m++) acc = cadd(acc, cmul(orow[m], bv[m]));
    out[q] = acc;
}

}  // namespace

extern "C" int laph_displace(laph_ctx_t c, const double *U, int dir, int sign, int length, const double *v, int n,
                             double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(U && v && out && v != out && n > 0, LAPH_EINVAL, "bad arguments");
    LAPH_CHECK(dir >= 0 && dir < 3 && (sign == 1 || sign == -1) && length >= 0, LAPH_EINVAL,
               "direction 0..2, sign +-1, length >= 0");
    const long total = (long)c->g.nt * c->g.V3;
    hipLaunchKernelGGL(k_displace, dim3(nblocks_for(total, kDisLanes)), dim3(kDisLanes), 0, c->stream, (const double2 *)U,
                       (const double2 *)v, (double2 *)out, c->g.ns, c->g.nt, n, dir, sign, length);
    LAPH_HIP(hipGetLastError());
    LAPH_API_END(c)
}

void overlap_slices(laph_ctx *c, const double2 *a, int na, const double2 *b, int nb, int k0, int k1, int k2,
                    double2 *phase, double2 *out, int parts)
{
    const long V3 = c->g.V3;
    LAPH_CHECK(parts >= 1 && V3 % (4L * parts) == 0, LAPH_EINVAL, "%d pieces of a slice", parts);
    hipLaunchKernelGGL(k_phase, dim3(nblocks_for(V3, 256)), dim3(256), 0, c->stream, phase, c->g.ns, k0, k1, k2);
    const int gn = (na + zg::kTM - 1) / zg::kTM, gm = (nb + zg::kTN - 1) / zg::kTN;
    LAPH_CHECK(gm <= 65535 && c->g.nt <= 65535, LAPH_EINVAL, "too many fields for one launch");
    LAPH_CHECK(3 * V3 < (1L << 31), LAPH_EINVAL, "slice too large");
    OverlapS os{a, b, phase, out, na, nb, (int)(3 * V3 / parts), gn, gm, (long)c->g.nt * parts, parts};
    LAPH_CHECK(zg::grid_of(os) < (1L << 31), LAPH_EINVAL, "too many fields for one launch");
    hipLaunchKernelGGL((zg::k_zgemm<12, true, true, OverlapS>), dim3((unsigned)zg::grid_of(os)), dim3(256), 0, c->stream, os);
    LAPH_HIP(hipGetLastError());
}

extern "C" int laph_mom_overlap(laph_ctx_t c, const double *a, int na, const double *b, int nb, const int *k,
                                double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(a && b && k && out && na > 0 && nb > 0, LAPH_EINVAL, "bad arguments");
    double2 *ph = (double2 *)ctx_named(c, "ovl.phase", sizeof(double2) * c->g.V3);
    overlap_slices(c, (const double2 *)a, na, (const double2 *)b, nb, k[0], k[1], k[2], ph, (double2 *)out);
    LAPH_API_END(c)
}

extern "C" int laph_overlap_apply(laph_ctx_t c, const double *O, int na, int nb, const double *b, int n, double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(O && b && out && b != out && na > 0 && nb > 0 && n > 0, LAPH_EINVAL, "bad arguments");
    const long nrt = (long)n * c->g.nt;
    hipLaunchKernelGGL(k_overlap_apply, dim3(nblocks_for(nrt * 4 * na, 256)), dim3(256), 0, c->stream,
                       (const double2 *)O, na, nb, (const double2 *)b, nrt, (double2 *)out, c->g.nt);
    LAPH_HIP(hipGetLastError());
    LAPH_API_END(c)
}
