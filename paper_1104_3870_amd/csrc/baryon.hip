// Baryon functions in LapH space (Sec. III.A: Eq. baryonfunc, and the baryon correlator
// of Eq. baryoncorr with its six noise orderings).
//
// With the trivial displacement every LapH-smeared quark sink is varphi = V_s f, so
//   B(t) = sum_{abg} c_abg sum_{n1 n2 n3} T[t][n1][n2][n3] f1[t][a][n1] f2[t][b][n2] f3[t][g][n3]
// with the eigenvector tensor T[t][n1][n2][n3] = sum_x e^{-ip.x} eps_abc V_n1(x,a) V_n2(x,b)
// V_n3(x,c) (totally antisymmetric: computed for n1 < n2 < n3, the rest by symmetry).  The
// contraction over (n1, n2, n3) for all dilution triples is three batched complex products:
//   X[n1 n2][k g]   = sum_n3 T[n1 n2][n3] F3[n3][k g]
//   Y[n1][j b][k g] = sum_n2 F2[n2][j b] X[n1 n2][k g]
//   Z[i a][j b k g] = sum_n1 F1[n1][i a] Y[n1][j b k g],   B[i][j][k] = sum c_abg Z[i a][j b][k g]
#include <algorithm>
#include <cmath>

#include "laph_impl.h"
#include "zgemm_mfma.h"

namespace {

// ------------------------------------------------------- batched complex product
// C[b](m, n) = sum_k op(A[b](m, k)) B[b](k, n), op = conj when conjA; every operand is
// addressed by strides (in complex elements); the batch index b splits into (b / nbi, b % nbi)
// with a stride per part.  Computed on the FP64 matrix cores (zgemm_mfma.h).
struct Zgemm {
    const double2 *A;
    long sAo, sAi, sAm, sAk;
    const double2 *B;
    long sBo, sBi, sBk, sBn;
    double2 *C;
    long sCo, sCi, sCm, sCn;
    int M, N, K, nbi, conjA;
};

struct GemmS {
    Zgemm g;
    int M, N, K;
    int tiles_m, tiles_n;
    long batches;
    __device__ zg::Side a(long bt) const
    {
        const long bo = bt / g.nbi, bi = bt - bo * g.nbi;
        return {g.A + bo * g.sAo + bi * g.sAi, g.sAm, g.sAk, M, g.conjA, nullptr};
    }
    __device__ zg::Side b(long bt) const
    {
        const long bo = bt / g.nbi, bi = bt - bo * g.nbi;
        return {g.B + bo * g.sBo + bi * g.sBi, g.sBn, g.sBk, N, 0, nullptr};
    }
    __device__ void store(long bt, int m, int n, double re, double im) const
    {
        const long bo = bt / g.nbi, bi = bt - bo * g.nbi;
        g.C[bo * g.sCo + bi * g.sCi + m * g.sCm + n * g.sCn] = make_double2(re, im);
    }
};

void zgemm(laph_ctx *c, const Zgemm &g, long batch)
{
    if (g.M <= 0 || g.N <= 0 || batch <= 0) return;
    const int gm = (g.M + zg::kTM - 1) / zg::kTM, gn = (g.N + zg::kTN - 1) / zg::kTN;
    GemmS s{g, g.M, g.N, g.K, gm, gn, batch};
    LAPH_CHECK(gn <= 65535 && batch <= 65535 && zg::grid_of(s) < (1L << 31), LAPH_EINVAL,
               "product too large for one launch");
    hipLaunchKernelGGL((zg::k_zgemm<8, false, false, GemmS>), dim3((unsigned)zg::grid_of(s)), dim3(256), 0, c->stream, s);
    LAPH_HIP(hipGetLastError());
}

// ------------------------------------------------------- eigenvector tensor
// X(a, b, c) = sum_x e^{-ip.x} (V_a(x) x V_b(x)) . V_c(x) for a < b < c as one product per
// slice: rows are the pairs (a, b), formed as cross products in the lanes that feed the
// matrix cores, columns the vectors c > b, K = 3 Ns^3.  Matrix and vector instructions share
// the FP64 pipe on gfx950 (measured: they add up), so the vector work per product is what
// this split keeps down: each row serves at least about N_v / 2 columns because the pairs
// are taken from the low side (b < N_v / 2, columns above b) and, by the mirror i -> N_v - 1
// - i, from the high side; 90% of the issued products are wanted at N_v = 112 (66% with one
// workgroup per first index).
//
// A workgroup's four waves take 16 pairs each and the same T <= kPT tiles of 16 columns.  K
// advances four sites a stage.  Lane l holds pair l % 16 at site l / 16: the three colours
// of its cross product are the A operands of three matrix steps (k = l / 16), so no A value
// passes through LDS.  Column vectors are staged in LDS (double-buffered, rows of 13 double2:
// conflict-free 16-byte reads), the next stage's loads in flight during the products.
//
// 24^3 x 128, N_v = 112: 190 ms (9.7e12 useful flops at 51 TFLOP/s, 58 TFLOP/s issued, of
// the 73 that back-to-back matrix instructions reach), 450 ms with one workgroup per first
// index, both operands staged through LDS.  At most 7 tiles: 4 and 5 (more workgroups per
// slice, each row formed more often) took 6% and 3% longer.
constexpr int kPT = 7;       // column tiles of 16 per workgroup
constexpr int kPS = 4;       // sites per stage
constexpr int kPR = 3 * kPS + 1;  // LDS row stride (double2)
// LDS rows of a stage: whole elements for all 256 lanes (rows past a tile count's own hold
// vectors nobody reads; a condition would sink the loads below the products)
constexpr int kPRows = ((kPT * 16 * 3 * kPS + 255) / 256 * 256 + 3 * kPS - 1) / (3 * kPS);
constexpr int kPBuf = kPRows * kPR;

// row r of the pairs a < b ordered by b
__host__ __device__ inline void pair_of(long r, int &a, int &b)
{
    int q = (int)((1.0 + sqrt(1.0 + 8.0 * (double)r)) * 0.5);
    while ((long)q * (q - 1) / 2 > r) q--;
    while ((long)(q + 1) * q / 2 <= r) q++;
    b = q;
    a = (int)(r - (long)q * (q - 1) / 2);
}

struct PairArgs {
    const double2 *V, *ph;
    double2 *out;
    int nv, nt, low;    // low: vectors on the low side, N_v / 2
    int blocks, chunks;  // workgroups per slice and side (pairs), column chunks
    int xcd;             // slices dealt to the XCDs in turn (nt a multiple of 8)
    long V3;
};

template <int T>
__device__ __forceinline__ void pair_tile(const PairArgs &P, double2 *lds, int t, int side, long row0, long rows,
                                          int ctop)
{
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, lr = l & 15, ls = l >> 4, nv = P.nv;
    const long K = 3 * P.V3;
    const double2 *Vt = P.V + (long)t * nv * K;
    auto vec = [&](int i) { return side ? nv - 1 - i : i; };
    // this lane's pair (past the end: the last one, not stored) and its site of a stage
    int a, b;
    pair_of(min(row0 + 16 * wave + lr, rows - 1), a, b);
    const double2 *pa = Vt + (long)vec(a) * K + 3 * ls, *pb = Vt + (long)vec(b) * K + 3 * ls, *pp = P.ph + ls;
    // this lane's staging elements: column row e / 12, element e % 12 of its 12 per stage
    constexpr int NB = (T * 16 * 3 * kPS + 255) / 256;
    const double2 *pc[NB];
    int dst[NB];
#pragma unroll
    for (int q = 0; q < NB; q++) {
        const int e = threadIdx.x + 256 * q, r = e / (3 * kPS), k = e - r * (3 * kPS);
        // column r of tile j is c = ctop - 16 (j + 1) + r % 16 (below 0: unused, any vector)
        const int c = ctop - 16 * (r / 16 + 1) + (r & 15);
        dst[q] = r * kPR + k;
        pc[q] = Vt + (long)vec(max(c, 0)) * K + k;
    }
    zg::d4 cr[T], ci[T];
#pragma unroll
    for (int j = 0; j < T; j++) {
        cr[j] = zg::d4{0.0, 0.0, 0.0, 0.0};
        ci[j] = zg::d4{0.0, 0.0, 0.0, 0.0};
    }
    double2 va[3], vb[3], vp, vc[NB];
    auto fetch = [&](long k) {  // the loads of stage k
#pragma unroll
        for (int c = 0; c < 3; c++) {
            va[c] = pa[3 * kPS * k + c];
            vb[c] = pb[3 * kPS * k + c];
        }
        vp = pp[kPS * k];
#pragma unroll
        for (int q = 0; q < NB; q++) vc[q] = pc[q][3 * kPS * k];
    };
    double xr[3], xi[3];
    auto put = [&](double2 *buf) {
#pragma unroll
        for (int q = 0; q < NB; q++) buf[dst[q]] = vc[q];
#pragma unroll
        for (int c = 0; c < 3; c++) va[c] = cmul(vp, va[c]);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
            xr[c] = va[c1].x * vb[c2].x - va[c1].y * vb[c2].y - va[c2].x * vb[c1].x + va[c2].y * vb[c1].y;
            xi[c] = va[c1].x * vb[c2].y + va[c1].y * vb[c2].x - va[c2].x * vb[c1].y - va[c2].y * vb[c1].x;
        }
    };
    fetch(0);
    put(lds);
    __syncthreads();
    const long stages = P.V3 / kPS;
    const double2 *base = lds + lr * kPR + 3 * ls;
    for (long k = 0; k < stages; k++) {
        const double2 *buf = base + (k & 1) * kPBuf;
        // (the last stage has nothing ahead of it and fetches its own again)
        fetch(min(k + 1, stages - 1));
#pragma unroll
        for (int c = 0; c < 3; c++) {
            double2 y[T];
#pragma unroll
            for (int j = 0; j < T; j++) y[j] = buf[j * 16 * kPR + c];
            const double ni = -xi[c];
#pragma unroll
            for (int j = 0; j < T; j++) {
                cr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[c], y[j].x, cr[j], 0, 0, 0);
                ci[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[c], y[j].y, ci[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < T; j++) {
                cr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ni, y[j].y, cr[j], 0, 0, 0);
                ci[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[c], y[j].x, ci[j], 0, 0, 0);
            }
        }
        put(lds + ((k + 1) & 1) * kPBuf);
        __syncthreads();
    }
    // element v of lane l: pair l / 16 + 4 v, column l % 16 of the tile
    const long nv2 = (long)nv * nv;
    double2 *out = P.out + (long)t * nv * nv2;
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const long r = row0 + 16 * wave + ls + 4 * v;
        if (r >= rows) continue;
        int ia, ib;
        pair_of(r, ia, ib);
        const long na = vec(ia), nb = vec(ib);
#pragma unroll
        for (int j = 0; j < T; j++) {
            const int ic = ctop - 16 * (j + 1) + lr;
            if (ic <= ib) continue;
            const long nc = vec(ic);
            const double2 q = make_double2(cr[j][v], ci[j][v]), mq = make_double2(-cr[j][v], -ci[j][v]);
            out[na * nv2 + nb * nv + nc] = q;
            out[nb * nv2 + nc * nv + na] = q;
            out[nc * nv2 + na * nv + nb] = q;
            out[na * nv2 + nc * nv + nb] = mq;
            out[nb * nv2 + na * nv + nc] = mq;
            out[nc * nv2 + nb * nv + na] = mq;
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_baryon_tensor_pairs(const PairArgs P)
{
    __shared__ double2 lds[2 * kPBuf];
    const int per = 2 * P.blocks * P.chunks;
    long g = blockIdx.x;
    int t;
    if (P.xcd) {  // workgroup g runs on XCD g % 8: a slice's workgroups share that XCD's L2
        const long q = g >> 3;
        t = (int)(q / per) * 8 + (int)(g & 7);
        g = q % per;
    } else {
        t = (int)(g / per);
        g -= (long)t * per;
    }
    const int chunk = (int)(g / (2 * P.blocks)), side = (int)(g & 1);
    const int h = side ? P.nv - P.low : P.low;
    const long row0 = 64 * ((g % (2 * P.blocks)) >> 1), rows = (long)h * (h - 1) / 2;
    if (row0 >= rows) return;
    // columns c > b of the workgroup's lowest b, in tiles of 16 from the top
    int a, b;
    pair_of(row0, a, b);
    const int need = (P.nv - 1 - b + 15) / 16, parts = (need + kPT - 1) / kPT, tc = (need + parts - 1) / parts;
    const int first = chunk * tc, T = min(tc, need - first);
    if (T <= 0) return;
    const int ctop = P.nv - 16 * first;
    switch (T) {
    case 1: pair_tile<1>(P, lds, t, side, row0, rows, ctop); break;
    case 2: pair_tile<2>(P, lds, t, side, row0, rows, ctop); break;
    case 3: pair_tile<3>(P, lds, t, side, row0, rows, ctop); break;
    case 4: pair_tile<4>(P, lds, t, side, row0, rows, ctop); break;
    case 5: pair_tile<5>(P, lds, t, side, row0, rows, ctop); break;
    case 6: pair_tile<6>(P, lds, t, side, row0, rows, ctop); break;
    default: pair_tile<7>(P, lds, t, side, row0, rows, ctop); break;
    }
}

__global__ void k_zero2(double2 *p, long n)
{
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (q < n) p[q] = make_double2(0.0, 0.0);
}

__global__ void k_phase3(double2 *ph, int ns, int k0, int k1, int k2)
{
    const long V3 = (long)ns * ns * ns;
    const long x = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (x >= V3) return;
    const int cx = (int)(x % ns), cy = (int)((x / ns) % ns), cz = (int)(x / ((long)ns * ns));
    const long m = (((long)k0 * cx + (long)k1 * cy + (long)k2 * cz) % ns + ns) % ns;
    double s, c;
    sincospi(-2.0 * (double)m / ns, &s, &c);
    ph[x] = make_double2(c, s);
}

// Ft[tl][n][i*4 + alpha] = f[i][t0 + tl][alpha][n] for tc slices
__global__ void k_coef_t(const double2 *__restrict__ f, int nf, int nt, int nv, int t0, int tc,
                         double2 *__restrict__ Ft)
{
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const long per = (long)nv * nf * 4;
    if (q >= tc * per) return;
    const int tl = (int)(q / per);
    const long r = q - tl * per;
    const int n = (int)(r / (nf * 4));
    const int ia = (int)(r - (long)n * nf * 4);
    const int i = ia / 4, a = ia % 4;
    Ft[q] = f[(((long)i * nt + t0 + tl) * 4 + a) * nv + n];
}

struct Spin64 {
    double2 c[64];
};

// B[t][i][j][k] = sum_{abg} c_abg Z[tl][(i a)][(j b)(k g)]
__global__ void k_spin3(Spin64 s, const double2 *__restrict__ Z, int n1, int n2, int n3, int t0, int tc,
                        double2 *__restrict__ out)
{
    const long q = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const long per = (long)n1 * n2 * n3;
    if (q >= tc * per) return;
    const int tl = (int)(q / per);
    const long r = q - tl * per;
    const int i = (int)(r / ((long)n2 * n3)), j = (int)((r / n3) % n2), k = (int)(r % n3);
    const long ncol = 16L * n2 * n3;
    const double2 *Zt = Z + (long)tl * (4L * n1) * ncol;
    double2 acc = make_double2(0.0, 0.0);
    for (int a = 0; a < 4; a++)
        for (int b = 0; b < 4; b++)
            for (int g = 0; g < 4; g++) {
                const double2 cc = s.c[(a * 4 + b) * 4 + g];
                if (cc.x == 0.0 && cc.y == 0.0) continue;
                acc = cadd(acc, cmul(cc, Zt[((long)i * 4 + a) * ncol + ((long)j * 4 + b) * (4L * n3) + k * 4 + g]));
            }
    out[(long)(t0 + tl) * per + r] = acc;
}

// C[tF] = sum_{b1 b2 b3} snk[tF][b1][b2][b3] conj(sum_s sign_s src[s][t0][b_s1][b_s2][b_s3]),
// the six orderings s of Eq. baryoncorr in a fixed order (noise order, sign)
__constant__ int kBPerm[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {2, 1, 0}, {1, 2, 0}, {2, 0, 1}};
__constant__ double kBSign[6] = {1, -1, -1, -1, 1, 1};

__global__ __launch_bounds__(256) void k_baryon_corr(const double2 *__restrict__ snk, const double2 *__restrict__ src,
                                                     int n, int nt, int t0, double2 *__restrict__ out)
{
    const int tf = blockIdx.x;
    const long n3 = (long)n * n * n;
    double2 acc = make_double2(0.0, 0.0);
    for (long q = threadIdx.x; q < n3; q += 256) {
        const int bidx[3] = {(int)(q / ((long)n * n)), (int)((q / n) % n), (int)(q % n)};
        double2 s = make_double2(0.0, 0.0);
        for (int p = 0; p < 6; p++) {
            const long idx = ((long)bidx[kBPerm[p][0]] * n + bidx[kBPerm[p][1]]) * n + bidx[kBPerm[p][2]];
            const double2 v = src[((long)p * nt + t0) * n3 + idx];
            s.x += kBSign[p] * v.x;
            s.y += kBSign[p] * v.y;
        }
        acc = cadd(acc, cconjmul(s, snk[(long)tf * n3 + q]));
    }
    __shared__ double2 red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = cadd(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[tf] = red[0];
}

}  // namespace

// slices per pass of laph_baryon_function: as many as fit a scratch budget of 1 GiB
static int baryon_chunk(int nt, int nv, int n1, int n2, int n3)
{
    const double per = 16.0 * ((double)nv * nv * 4 * n3 + (double)nv * 16 * n2 * n3 + 4.0 * n1 * 16 * n2 * n3 +
                               4.0 * nv * (n1 + n2 + n3));
    int tc = (int)std::max(1.0, std::floor((double)(1u << 30) / per));
    return std::min(tc, nt);
}

size_t baryon_scratch_bytes(const Geom &g, int nv, int n1, int n2, int n3)
{
    const long tc = baryon_chunk(g.nt, nv, n1, n2, n3);
    return ws_align(16 * tc * nv * 4 * n1) + ws_align(16 * tc * nv * 4 * n2) + ws_align(16 * tc * nv * 4 * n3) +
           ws_align(16 * tc * nv * nv * 4 * n3) + ws_align(16 * tc * nv * 16 * n2 * n3) +
           ws_align(16 * tc * 4 * n1 * 16 * n2 * n3);
}

extern "C" int laph_baryon_tensor(laph_ctx_t c, const double *evecs, int nv, const int *k, double *T)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(evecs && k && T && nv > 0, LAPH_EINVAL, "bad arguments");
    const long V3 = c->g.V3;
    double2 *ph = (double2 *)ctx_named(c, "bar.phase", sizeof(double2) * V3);
    hipLaunchKernelGGL(k_phase3, dim3(nblocks_for(V3, 256)), dim3(256), 0, c->stream, ph, c->g.ns, k[0], k[1], k[2]);
    LAPH_CHECK(nv <= 416, LAPH_EINVAL, "nv too large");
    LAPH_CHECK(c->g.nt <= 65535 && 3 * V3 < (1L << 31), LAPH_EINVAL, "lattice too large for one launch");
    const long total = (long)c->g.nt * nv * nv * nv;
    hipLaunchKernelGGL(k_zero2, dim3(nblocks_for(total, 256)), dim3(256), 0, c->stream, (double2 *)T, total);
    const int low = nv / 2, high = nv - low, nt = c->g.nt;
    const long pairs = (long)high * (high - 1) / 2;
    if (pairs > 0) {
        PairArgs P{(const double2 *)evecs, (const double2 *)ph, (double2 *)T, nv, nt, low, (int)((pairs + 63) / 64),
                   ((nv + 15) / 16 + kPT - 1) / kPT, nt % 8 == 0, V3};
        const long blocks = (long)nt * 2 * P.blocks * P.chunks;
        LAPH_CHECK(blocks < (1L << 31), LAPH_EINVAL, "too many workgroups for one launch");
        hipLaunchKernelGGL(k_baryon_tensor_pairs, dim3((unsigned)blocks), dim3(256), 0, c->stream, P);
    }
    LAPH_HIP(hipGetLastError());
    LAPH_API_END(c)
}

extern "C" int laph_baryon_function(laph_ctx_t c, const double *T, int nv, const double *cs, const double *f1, int n1,
                                    const double *f2, int n2, const double *f3, int n3, double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(T && cs && f1 && f2 && f3 && out && nv > 0 && n1 > 0 && n2 > 0 && n3 > 0, LAPH_EINVAL,
               "bad arguments");
    Spin64 s;
    for (int q = 0; q < 64; q++) {
        LAPH_CHECK(std::isfinite(cs[2 * q]) && std::isfinite(cs[2 * q + 1]), LAPH_EINVAL, "spin tensor not finite");
        s.c[q] = make_double2(cs[2 * q], cs[2 * q + 1]);
    }
    const int nt = c->g.nt;
    const int tc = baryon_chunk(nt, nv, n1, n2, n3);
    const long c1 = 4L * n1, c2 = 4L * n2, c3 = 4L * n3;
    double2 *F1 = (double2 *)ctx_named(c, "bar.F1", 16 * (size_t)tc * nv * c1);
    double2 *F2 = (double2 *)ctx_named(c, "bar.F2", 16 * (size_t)tc * nv * c2);
    double2 *F3 = (double2 *)ctx_named(c, "bar.F3", 16 * (size_t)tc * nv * c3);
    double2 *X = (double2 *)ctx_named(c, "bar.X", 16 * (size_t)tc * nv * nv * c3);
    double2 *Y = (double2 *)ctx_named(c, "bar.Y", 16 * (size_t)tc * nv * c2 * c3);
    double2 *Z = (double2 *)ctx_named(c, "bar.Z", 16 * (size_t)tc * c1 * c2 * c3);
    const double2 *Td = (const double2 *)T;
    for (int t0 = 0; t0 < nt; t0 += tc) {
        const int tcn = std::min(tc, nt - t0);
        hipLaunchKernelGGL(k_coef_t, dim3(nblocks_for((long)tcn * nv * c1, 256)), dim3(256), 0, c->stream,
                           (const double2 *)f1, n1, nt, nv, t0, tcn, F1);
        hipLaunchKernelGGL(k_coef_t, dim3(nblocks_for((long)tcn * nv * c2, 256)), dim3(256), 0, c->stream,
                           (const double2 *)f2, n2, nt, nv, t0, tcn, F2);
        hipLaunchKernelGGL(k_coef_t, dim3(nblocks_for((long)tcn * nv * c3, 256)), dim3(256), 0, c->stream,
                           (const double2 *)f3, n3, nt, nv, t0, tcn, F3);
        LAPH_HIP(hipGetLastError());
        // X[tl][n1 n2][k g] = sum_n3 T[t][n1 n2][n3] F3[tl][n3][k g]
        Zgemm gx{Td + (size_t)t0 * nv * nv * nv, (long)nv * nv * nv, 0, nv, 1,
                 F3, nv * c3, 0, c3, 1,
                 X, (long)nv * nv * c3, 0, c3, 1,
                 nv * nv, (int)c3, nv, 1, 0};
        zgemm(c, gx, tcn);
        // Y[tl][n1][j b][k g] = sum_n2 F2[tl][n2][j b] X[tl][n1 n2][k g]
        Zgemm gy{F2, nv * c2, 0, 1, c2,
                 X, (long)nv * nv * c3, (long)nv * c3, c3, 1,
                 Y, (long)nv * c2 * c3, c2 * c3, c3, 1,
                 (int)c2, (int)c3, nv, nv, 0};
        zgemm(c, gy, (long)tcn * nv);
        // Z[tl][i a][(j b)(k g)] = sum_n1 F1[tl][n1][i a] Y[tl][n1][(j b)(k g)]
        Zgemm gz{F1, nv * c1, 0, 1, c1,
                 Y, (long)nv * c2 * c3, 0, c2 * c3, 1,
                 Z, c1 * c2 * c3, 0, c2 * c3, 1,
                 (int)c1, (int)(c2 * c3), nv, 1, 0};
        zgemm(c, gz, tcn);
        const long nout = (long)tcn * n1 * n2 * n3;
        hipLaunchKernelGGL(k_spin3, dim3(nblocks_for(nout, 256)), dim3(256), 0, c->stream, s, (const double2 *)Z, n1,
                           n2, n3, t0, tcn, (double2 *)out);
        LAPH_HIP(hipGetLastError());
    }
    LAPH_API_END(c)
}

extern "C" int laph_baryon_correlator(laph_ctx_t c, const double *snk, const double *src, int n, int t0, double *out)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(snk && src && out && n > 0, LAPH_EINVAL, "bad arguments");
    LAPH_CHECK(t0 >= 0 && t0 < c->g.nt, LAPH_EINVAL, "t0 out of range");
    hipLaunchKernelGGL(k_baryon_corr, dim3(c->g.nt), dim3(256), 0, c->stream, (const double2 *)snk,
                       (const double2 *)src, n, c->g.nt, t0, (double2 *)out);
    LAPH_HIP(hipGetLastError());
    LAPH_API_END(c)
}
