// laph_eigvecs: the N_v lowest eigenpairs of -Lap on every time slice by the
// Krylov-spectral restarted (thick-restart) Lanczos method of Sec. IV, batched over all
// slices so that one launch works on every slice at once.
//
//  * operator A = T_n(B), B = 1 + 2/(lamL - lamC)(Lap + lamC): the wanted low end of
//    -Lap becomes the top of A;
//  * the local three-term part is subtracted first, then full global reorthogonalisation
//    by classical Gram-Schmidt; a pass is repeated while it shrinks the vector by more than
//    1/kappa, kappa = sqrt(2), at most four repeats;
//  * Rayleigh-Ritz on the projected (real symmetric) matrix by parallel cyclic Jacobi,
//    one workgroup per slice;
//  * a Ritz pair with |A y - theta y| = beta_m |e_m^T s| < tol |A| is locked (kept in
//    the basis for orthogonalisation only); |A| is the largest |theta| seen;
//  * after a restart R_tot = N_v + (m - N_v)/2 vectors remain (locked + best Ritz
//    vectors) and the residual vector continues the Krylov sequence (this restart size
//    is our reading of the rule the paper takes from Wu and Simon; it bounds the kept
//    count by the converged count below and by m - locked - 12 above).
// Eigenvalues are Rayleigh quotients on -Lap; each eigenvector gets the phase that makes
// its first component with modulus >= 0.1 of the maximum real and positive.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <type_traits>

#include "laplace.h"

namespace {

__device__ __forceinline__ uint4 philox10(uint4 c, uint2 k)
{
#pragma unroll
    for (int r = 0; r < 10; r++) {
        uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
        uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
        c = make_uint4(hi1 ^ c.y ^ k.x, lo1, hi0 ^ c.w ^ k.y, lo0);
        k.x += 0x9E3779B9u;
        k.y += 0xBB67AE85u;
    }
    return c;
}

// --------------------------------------------------------------- Gram-Schmidt
// One step takes w = A q_j to q_{j+1}: the local part alpha q_j + beta q_{j-1} of the
// three-term recurrence (alpha = <q_j, w>, beta the last norm) is subtracted first, and the
// full pass c = Q^dag w, w -= Q c over the whole basis then removes what rounding and the
// kept Ritz vectors of a restart leave.  A further full pass follows while one shrinks the
// vector by more than 1 / kappa.  Both kernels of a pass stream the basis once and are bound
// by HBM: a workgroup takes tiles of 32 rows x cnt columns, lane (row r, column group g)
// holding columns g, g + 8, ... of its row in registers, so that a tile's up to 20 loads of
// 16 bytes per lane are in flight together.  Measured on 16 slices of 24^3, 137-160 columns
// (1.57 GB on average): dots 296 us and update 279 us, 5.3 and 5.6 TB/s.  Two full passes
// per step without the local part, the dots one column per wave, took 1.82 ms per step with
// their 27 small launches; a step's Gram-Schmidt now takes 0.62 ms in five launches.
constexpr int kGsRows = 32, kGsGroups = 8;
constexpr double kKappa = 1.4142135623730951;

// columns per lane for cnt columns, as a template argument
template <class F>
void gs_columns(int cnt, F f)
{
    if (cnt <= 5 * kGsGroups)
        f(std::integral_constant<int, 5>());
    else if (cnt <= 10 * kGsGroups)
        f(std::integral_constant<int, 10>());
    else if (cnt <= 15 * kGsGroups)
        f(std::integral_constant<int, 15>());
    else
        f(std::integral_constant<int, 20>());
}

template <int NC>
__device__ __forceinline__ void gs_tile(const double2 *__restrict__ Q, long n, int cnt, int g, long row,
                                        double2 (&q)[NC])
{
#pragma unroll
    for (int i = 0; i < NC; i++) {
        const int a = g + kGsGroups * i;
        q[i] = make_double2(0.0, 0.0);
        if (row < n && a < cnt) q[i] = Q[(long)a * n + row];
    }
}

// block-wide sum of one double per lane (red: one value per wave)
__device__ __forceinline__ double block_sum(double v, double *red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < (int)(blockDim.x >> 6); k++) s += red[k];
    return s;
}

// partial[t][block][a] = the block's part of <q_a, w'>, wpart[t][block] of |w'|^2, with w' = w
// (LOCAL = false) or w' = w - alpha q_j - beta q_{j-1}, written to wout; alpha and
// |w|^2 come from the Laplacian's block sums lsum[t][nl][3], beta = T[j-1][j]
template <int NC, bool LOCAL>
__global__ __launch_bounds__(256) void k_gs_dots(const double2 *__restrict__ Qall, long qslice, long n,
                                                 const double2 *__restrict__ w, double2 *__restrict__ wout, int cnt,
                                                 const double *__restrict__ lsum, int nl, const double *__restrict__ T,
                                                 int m, double *__restrict__ alpha, double *__restrict__ nb0,
                                                 double2 *__restrict__ partial, int pstride,
                                                 double *__restrict__ wpart)
{
    __shared__ double red[4];
    const int t = blockIdx.y, r = threadIdx.x & (kGsRows - 1), g = threadIdx.x / kGsRows, j = cnt - 1;
    const double2 *Q = Qall + t * qslice;
    double2 al = make_double2(0.0, 0.0);
    double be = 0.0;
    if (LOCAL) {
        double s0 = 0, s1 = 0, s2 = 0;
        for (int k = threadIdx.x; k < nl; k += 256) {
            const double *p = lsum + ((long)t * nl + k) * 3;
            s0 += p[0];
            s1 += p[1];
            s2 += p[2];
        }
        al = make_double2(block_sum(s0, red), block_sum(s1, red));
        const double nn = block_sum(s2, red);
        if (j > 0) be = T[((long)t * m + j - 1) * m + j];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            alpha[t] = al.x;
            nb0[t] = sqrt(nn);
        }
    }
    double2 acc[NC];
#pragma unroll
    for (int i = 0; i < NC; i++) acc[i] = make_double2(0.0, 0.0);
    double nrm = 0.0;
    for (long tile = blockIdx.x; tile * kGsRows < n; tile += gridDim.x) {
        const long row = tile * kGsRows + r;
        double2 q[NC], v = make_double2(0.0, 0.0);
        gs_tile<NC>(Q, n, cnt, g, row, q);
        if (row < n) {
            v = w[t * n + row];
            if (LOCAL) {
                v = csub(v, cmul(al, Q[(long)j * n + row]));
                if (j > 0) v = csub(v, cscale(Q[(long)(j - 1) * n + row], be));
                if (g == 0) wout[t * n + row] = v;
            }
        }
#pragma unroll
        for (int i = 0; i < NC; i++) {
            acc[i].x += q[i].x * v.x + q[i].y * v.y;
            acc[i].y += q[i].x * v.y - q[i].y * v.x;
        }
        if (g == 0) nrm += cnorm2(v);
    }
#pragma unroll
    for (int i = 0; i < NC; i++) {
        for (int o = kGsRows / 2; o > 0; o >>= 1) {
            acc[i].x += __shfl_down(acc[i].x, o, kGsRows);
            acc[i].y += __shfl_down(acc[i].y, o, kGsRows);
        }
        const int a = g + kGsGroups * i;
        if (r == 0 && a < cnt) partial[((long)t * gridDim.x + blockIdx.x) * pstride + a] = acc[i];
    }
    nrm = block_sum(nrm, red);
    if (threadIdx.x == 0) wpart[(long)t * gridDim.x + blockIdx.x] = nrm;
}

// coef[t][a] = the block sums of <q_a, w>, nb[t] = |w|; T[t][a][j] for a in [nlock[t], j]: the
// coefficient, plus what the column holds (accumulate) or the local part (alpha on the
// diagonal, beta, still in its place, above it)
__global__ void k_gs_fin(const double2 *__restrict__ partial, const double *__restrict__ wpart, int nblk, int pstride,
                         int cnt, double2 *__restrict__ coef, double *__restrict__ nb, const double *__restrict__ alpha,
                         double *__restrict__ T, int m, const int *__restrict__ nlock, int accumulate)
{
    __shared__ double red[4];
    const int t = blockIdx.x, j = cnt - 1;
    for (int a = threadIdx.x; a < cnt; a += blockDim.x) {
        double2 s = make_double2(0, 0);
        for (int k = 0; k < nblk; k++) s = cadd(s, partial[((long)t * nblk + k) * pstride + a]);
        coef[(long)t * pstride + a] = s;
        if (a >= nlock[t]) {
            double *e = T + ((long)t * m + a) * m + j;
            const double had = accumulate || a == j - 1 ? *e : a == j ? alpha[t] : 0.0;
            *e = had + s.x;
        }
    }
    double s = 0.0;
    for (int k = threadIdx.x; k < nblk; k += blockDim.x) s += wpart[(long)t * nblk + k];
    s = block_sum(s, red);
    if (threadIdx.x == 0) nb[t] = sqrt(s);
}

// w[t] -= sum_a q_a coef[t][a];  npart[t][block] the block's part of |w|^2
template <int NC>
__global__ __launch_bounds__(256) void k_gs_update(const double2 *__restrict__ Qall, long qslice, long n,
                                                   double2 *__restrict__ w, int cnt, const double2 *__restrict__ coef,
                                                   int pstride, double *__restrict__ npart)
{
    __shared__ double2 cs[kGsGroups * NC], part[2][kGsGroups][kGsRows];
    __shared__ double red[4];
    const int t = blockIdx.y, r = threadIdx.x & (kGsRows - 1), g = threadIdx.x / kGsRows;
    const double2 *Q = Qall + t * qslice;
    for (int a = threadIdx.x; a < kGsGroups * NC; a += 256)
        cs[a] = a < cnt ? coef[(long)t * pstride + a] : make_double2(0.0, 0.0);
    __syncthreads();
    double nrm = 0.0;
    int buf = 0;
    for (long tile = blockIdx.x; tile * kGsRows < n; tile += gridDim.x, buf ^= 1) {
        const long row = tile * kGsRows + r;
        double2 q[NC], s = make_double2(0.0, 0.0), v = s;
        gs_tile<NC>(Q, n, cnt, g, row, q);
        if (g == 0 && row < n) v = w[t * n + row];
#pragma unroll
        for (int i = 0; i < NC; i++) s = cadd(s, cmul(q[i], cs[g + kGsGroups * i]));
        part[buf][g][r] = s;
        __syncthreads();  // the other half of part is written before the next one is read
        if (g == 0 && row < n) {
#pragma unroll
            for (int k = 0; k < kGsGroups; k++) v = csub(v, part[buf][k][r]);
            w[t * n + row] = v;
            nrm += cnorm2(v);
        }
    }
    nrm = block_sum(nrm, red);
    if (threadIdx.x == 0) npart[(long)t * gridDim.x + blockIdx.x] = nrm;
}

// After a step's full passes: nrm[t] = |w| and T[j][j+1] = |w| (beta_out at the last step).
// Two rare cases are dealt with here, one workgroup for the slice: a pass that shrank the
// vector by more than 1 / kappa is repeated (at most until five passes are done), and where |w| fell
// below 1e-10 of |A q_j| (an invariant subspace) a fresh Philox vector, orthogonalised
// twice, takes its place with T[j][j+1] = 0.
__global__ __launch_bounds__(1024) void k_gs_check(const double2 *__restrict__ Qall, long qslice, long n,
                                                   double2 *__restrict__ wall, int cnt,
                                                   const double *__restrict__ npart, int nblk,
                                                   const double *__restrict__ nb, const double *__restrict__ nb0,
                                                   double *__restrict__ T, int m, const int *__restrict__ nlock,
                                                   int passes, uint32_t seed, double *__restrict__ nrm,
                                                   double *__restrict__ beta_out)
{
    __shared__ double2 cf[160];
    __shared__ double red[16];
    const int t = blockIdx.x, j = cnt - 1, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double2 *Q = Qall + t * qslice;
    double2 *w = wall + t * n;
    auto pass = [&](bool intoT) {
        for (int a = wave; a < cnt; a += 16) {
            double re = 0, im = 0;
            for (long row = lane; row < n; row += 64) {
                const double2 u = Q[(long)a * n + row], v = w[row];
                re += u.x * v.x + u.y * v.y;
                im += u.x * v.y - u.y * v.x;
            }
            for (int o = 32; o > 0; o >>= 1) {
                re += __shfl_down(re, o, 64);
                im += __shfl_down(im, o, 64);
            }
            if (lane == 0) cf[a] = make_double2(re, im);
        }
        __syncthreads();
        if (intoT)
            for (int a = threadIdx.x; a < cnt; a += 1024)
                if (a >= nlock[t]) T[((long)t * m + a) * m + j] += cf[a].x;
        double s = 0.0;
        for (long row = threadIdx.x; row < n; row += 1024) {
            double2 v = w[row];
            for (int a = 0; a < cnt; a++) v = csub(v, cmul(Q[(long)a * n + row], cf[a]));
            w[row] = v;
            s += cnorm2(v);
        }
        return sqrt(block_sum(s, red));  // (a barrier: w and cf are whole for the next pass)
    };
    double s = 0.0;
    for (int k = threadIdx.x; k < nblk; k += 1024) s += npart[(long)t * nblk + k];
    double v = sqrt(block_sum(s, red)), before = nb[t];
    for (; v < before / kKappa && passes < 5; passes++) {
        before = v;
        v = pass(true);
    }
    double link = v;
    if (!(v > 1e-10 * nb0[t])) {
        for (long row = threadIdx.x; row < n; row += 1024) {
            const uint4 p = philox10(make_uint4((uint32_t)row, (uint32_t)t, (uint32_t)j, 0x42524bu),
                                     make_uint2(seed, 0x4C5A4E43u));
            w[row] = make_double2(p.x * 2.3283064365386963e-10 - 0.5, p.y * 2.3283064365386963e-10 - 0.5);
        }
        __syncthreads();
        pass(false);
        v = pass(false);
        link = 0.0;
    }
    if (threadIdx.x == 0) {
        nrm[t] = v;
        if (j + 1 < m) T[((long)t * m + j) * m + j + 1] = link;
        if (beta_out) beta_out[t] = link;
    }
}

// q[t] = w[t] / nrm[t]
__global__ __launch_bounds__(256) void k_gs_scale(const double2 *__restrict__ w, long n, double2 *__restrict__ q,
                                                  long qslice, const double *__restrict__ nrm)
{
    const int t = blockIdx.y;
    const long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (row < n) q[t * qslice + row] = cscale(w[t * n + row], 1.0 / nrm[t]);
}

// pieces the Gram matrices' sums over a slice's sites are taken in, of 64 sites or more: one sum
// after the other over all 3 Ns^3 terms puts their rounding into the result, which on plane
// waves, terms all of one size, goes one way (24^3, N_v = 112: 1.2e-12 reported for vectors
// orthonormal to 4.7e-13)
int gram_parts(long V3)
{
    long d = std::max(1L, V3 / 64);
    while ((V3 / 4) % d) d--;
    return (int)d;
}

// dev[t][block] = max over the block's share of (a, p) of |O[t][a][p] - delta_ap| for the Gram
// matrices given in pieces, O [nt][parts][nv][nv]
__global__ __launch_bounds__(256) void k_gram_dev(const double2 *__restrict__ O, int nv, int parts,
                                                  double *__restrict__ dev)
{
    __shared__ double red[256];
    const int t = blockIdx.y;
    double mx = 0.0;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < nv * nv; e += 256 * gridDim.x) {
        double2 v = make_double2(0.0, 0.0);
        for (int q = 0; q < parts; q++) v = cadd(v, O[((long)t * parts + q) * nv * nv + e]);
        if (e / nv == e % nv) v.x -= 1.0;
        mx = fmax(mx, sqrt(cnorm2(v)));
    }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) dev[(long)t * gridDim.x + blockIdx.x] = red[0];
}

// partial |w|^2 (no update)
__global__ __launch_bounds__(256) void k_norm_slices(const double2 *__restrict__ w, long wslice, long n,
                                                     double *__restrict__ npart)
{
    int t = blockIdx.y;
    __shared__ double red[256];
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    red[threadIdx.x] = row < n ? cnorm2(w[t * wslice + row]) : 0.0;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) npart[(long)t * gridDim.x + blockIdx.x] = red[0];
}

// nrm[t] = sqrt of the sum of a slice's block sums
__global__ __launch_bounds__(256) void k_norm_fin(const double *__restrict__ npart, int nblk, double *__restrict__ nrm)
{
    __shared__ double red[4];
    const int t = blockIdx.x;
    double s = 0;
    for (int b = threadIdx.x; b < nblk; b += 256) s += npart[(long)t * nblk + b];
    s = block_sum(s, red);
    if (threadIdx.x == 0) nrm[t] = sqrt(s);
}

__global__ __launch_bounds__(256) void k_random(double2 *__restrict__ q, long qslice, long n, uint32_t seed)
{
    int t = blockIdx.y;
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n) return;
    uint4 r = philox10(make_uint4((uint32_t)row, (uint32_t)t, 0u, 0x53545254u), make_uint2(seed, 0x4C5A4E43u));
    q[t * qslice + row] = make_double2(r.x * 2.3283064365386963e-10 - 0.5, r.y * 2.3283064365386963e-10 - 0.5);
}

__global__ __launch_bounds__(256) void k_scale(double2 *__restrict__ q, long qslice, long n, const double *nrm)
{
    int t = blockIdx.y;
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (row < n) q[t * qslice + row] = cscale(q[t * qslice + row], 1.0 / nrm[t]);
}

// ------------------------------------------------------------- Rayleigh-Ritz
// Parallel cyclic Jacobi on the na x na active block of T (na = m - nlock <= 160), one
// workgroup per slice.  The symmetric matrix stays in LDS for whole sweeps: only its upper
// triangle, folded into na/2 rows of na + 1 doubles (103 KB at na = 160, where the square
// would need 205 of the 160 KB).  A round of disjoint pairs (p_k, q_k) splits the matrix
// into 2 x 2 blocks (pair k, pair l), each owned by one lane, which applies both rotations
// at once; so a round takes two barriers.  The rotations are written out, and
// k_jacobi_vectors applies them to the rows of the eigenvector matrix, which are
// independent of each other and so spread over many workgroups.  Both are bound by the
// latency of a round (rotation, barrier, LDS pass).  Per restart at m = 160 (16 slices of
// 24^3): 1.4 + 0.5 ms, against 34.8 ms for one workgroup of 256 lanes with both matrices in
// global memory.
constexpr int kJacLanes = 1024;
constexpr int kJacRows = 16;    // eigenvector rows per workgroup
constexpr int kJacSweeps = 40;  // most sweeps of one Rayleigh-Ritz step

// element (i, j) of a symmetric N x N matrix (N even) in the folded upper triangle: rows
// below N / 2 keep their place, row i of the rest fills the free start of row N - 1 - i
__device__ __forceinline__ int fold(int i, int j, int N)
{
    const int lo = min(i, j), hi = max(i, j);
    return lo < (N >> 1) ? lo * (N + 1) + hi + 1 : (N - 1 - lo) * (N + 1) + N - 1 - hi;
}

// pair k of a round: every index meets every other once in the N - 1 rounds of a sweep
__device__ __forceinline__ void jacobi_pair(int k, int round, int N, int &p, int &q)
{
    if (k == 0) {
        p = N - 1;
        q = round;
        return;
    }
    p = round + k;
    if (p >= N - 1) p -= N - 1;
    q = round - k;
    if (q < 0) q += N - 1;
}

// M[t] = the active block of T (rows and columns nlock..m-1, symmetric, from its upper
// triangle) in folded form, padded by a zero row when na is odd; done[t] = 0
__global__ void k_active(const double *__restrict__ T, double *__restrict__ M, int m, const int *__restrict__ nlock,
                         int *__restrict__ done)
{
    const int t = blockIdx.x, l = nlock[t], na = m - l, N = na + (na & 1);
    for (int idx = threadIdx.x; idx < N * N; idx += blockDim.x) {
        const int i = idx / N, j = idx - i * N;
        if (i > j) continue;
        M[(long)t * m * m + fold(i, j, N)] = j < na ? T[((long)t * m + l + i) * m + l + j] : 0.0;
    }
    if (threadIdx.x == 0) done[t] = 0;
}

// up to `most` sweeps on M[t]; rot[t][(sweep * (N - 1) + round) * (N / 2) + k] = (c, s) of
// pair k, nsw[t] the sweeps done here, done[t] = 1 once the off-diagonal norm is below
// 1e-15 of the whole
__global__ __launch_bounds__(kJacLanes) void k_jacobi_sweeps(double *__restrict__ Mall, double2 *__restrict__ rot,
                                                             long rstride, int m, const int *__restrict__ nlock,
                                                             int most, int *__restrict__ nsw, int *__restrict__ done)
{
    extern __shared__ __attribute__((aligned(16))) double A[];
    const int t = blockIdx.x, na = m - nlock[t], N = na + (na & 1), h = N >> 1, size = h * (N + 1);
    double2 *cs = (double2 *)(A + size + (size & 1));
    __shared__ double red[2][kJacLanes / 64];
    __shared__ int stop;
    if (done[t]) {
        if (threadIdx.x == 0) nsw[t] = 0;
        return;
    }
    double *M = Mall + (long)t * m * m;
    double2 *rt = rot + t * rstride;
    for (int e = threadIdx.x; e < size; e += kJacLanes) A[e] = M[e];
    // this lane's 2 x 2 blocks (k < l), the same ones in every round
    constexpr int kOwn = (80 * 79 / 2 + kJacLanes - 1) / kJacLanes;
    int bk[kOwn], bl[kOwn];
#pragma unroll
    for (int o = 0; o < kOwn; o++) {
        const int b = threadIdx.x + o * kJacLanes;
        int l = (int)((1.0f + sqrtf(1.0f + 8.0f * b)) * 0.5f);
        while (l * (l - 1) / 2 > b) l--;
        while ((l + 1) * l / 2 <= b) l++;
        bl[o] = l < h ? l : -1;
        bk[o] = b - l * (l - 1) / 2;
    }
    int sweep = 0;
    for (;; sweep++) {
        __syncthreads();
        double off = 0, tot = 0;
        for (int e = threadIdx.x; e < size; e += kJacLanes) {
            const int r = e / (N + 1), c = e - r * (N + 1);
            const bool dia = c > r ? c - 1 == r : N - 1 - c == N - 1 - r;
            const double v = A[e] * A[e];
            tot += dia ? v : 2 * v;
            if (!dia) off += 2 * v;
        }
        for (int w = 32; w > 0; w >>= 1) {
            off += __shfl_down(off, w, 64);
            tot += __shfl_down(tot, w, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            red[0][threadIdx.x >> 6] = off;
            red[1][threadIdx.x >> 6] = tot;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double so = 0, st = 0;
            for (int w = 0; w < kJacLanes / 64; w++) {
                so += red[0][w];
                st += red[1][w];
            }
            stop = so <= 1e-30 * st;
        }
        __syncthreads();
        if (stop || sweep == most) break;
        for (int round = 0; round < N - 1; round++) {
            if ((int)threadIdx.x < h) {
                int p, q;
                jacobi_pair(threadIdx.x, round, N, p, q);
                const int ipq = fold(p, q, N), ip = fold(p, p, N), iq = fold(q, q, N);
                const double apq = A[ipq];
                double c = 1, sn = 0;
                if (fabs(apq) > 1e-300) {
                    const double app = A[ip], aqq = A[iq];
                    const double tau = (aqq - app) / (2 * apq);
                    const double tt = (tau >= 0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1 + tau * tau));
                    c = 1 / sqrt(1 + tt * tt);
                    sn = tt * c;
                    A[ip] = app - tt * apq;
                    A[iq] = aqq + tt * apq;
                    A[ipq] = 0.0;
                }
                cs[threadIdx.x] = make_double2(c, sn);
                rt[((long)sweep * (N - 1) + round) * h + threadIdx.x] = make_double2(c, sn);
            }
            __syncthreads();
#pragma unroll
            for (int o = 0; o < kOwn; o++) {
                if (bl[o] < 0) continue;
                int pk, qk, pl, ql;
                jacobi_pair(bk[o], round, N, pk, qk);
                jacobi_pair(bl[o], round, N, pl, ql);
                const int i11 = fold(pk, pl, N), i12 = fold(pk, ql, N), i21 = fold(qk, pl, N), i22 = fold(qk, ql, N);
                const double2 ck = cs[bk[o]], cl = cs[bl[o]];
                const double a11 = A[i11], a12 = A[i12], a21 = A[i21], a22 = A[i22];
                const double r11 = ck.x * a11 - ck.y * a21, r12 = ck.x * a12 - ck.y * a22;
                const double r21 = ck.y * a11 + ck.x * a21, r22 = ck.y * a12 + ck.x * a22;
                A[i11] = cl.x * r11 - cl.y * r12;
                A[i12] = cl.y * r11 + cl.x * r12;
                A[i21] = cl.x * r21 - cl.y * r22;
                A[i22] = cl.y * r21 + cl.x * r22;
            }
            __syncthreads();
        }
    }
    for (int e = threadIdx.x; e < size; e += kJacLanes) M[e] = A[e];
    if (threadIdx.x == 0) {
        nsw[t] = sweep;
        done[t] = stop;
    }
}

// Y[t] <- Y[t] J for the sweeps k_jacobi_sweeps recorded (first: Y[t] starts as the unit
// matrix); kJacRows rows per workgroup in LDS, the next round's rotations loaded during
// the current one
__global__ __launch_bounds__(256) void k_jacobi_vectors(double *__restrict__ Yall, const double2 *__restrict__ rot,
                                                        long rstride, int m, const int *__restrict__ nlock,
                                                        const int *__restrict__ nsw, int first)
{
    __shared__ double Y[kJacRows][161];
    __shared__ double2 cs[2][80];
    const int t = blockIdx.y, na = m - nlock[t], N = na + (na & 1), h = N >> 1, r0 = blockIdx.x * kJacRows;
    const int sweeps = nsw[t];
    if (r0 >= na || (!sweeps && !first)) return;
    double *Yg = Yall + (long)t * m * m;
    const double2 *rt = rot + t * rstride;
    for (int e = threadIdx.x; e < kJacRows * N; e += 256) {
        const int r = e / N, c = e - r * N;
        double v = r0 + r == c ? 1.0 : 0.0;
        if (!first && r0 + r < na && c < na) v = Yg[(long)(r0 + r) * m + c];
        Y[r][c] = v;
    }
    const int rounds = sweeps * (N - 1), row = threadIdx.x & (kJacRows - 1), slot = threadIdx.x / kJacRows;
    double2 nx = make_double2(1.0, 0.0);
    if ((int)threadIdx.x < h && rounds > 0) nx = rt[threadIdx.x];
    int round = 0;
    for (int g = 0; g < rounds; g++) {
        if ((int)threadIdx.x < h) {
            cs[g & 1][threadIdx.x] = nx;
            if (g + 1 < rounds) nx = rt[(long)(g + 1) * h + threadIdx.x];
        }
        __syncthreads();
        for (int k = slot; k < h; k += 256 / kJacRows) {
            int p, q;
            jacobi_pair(k, round, N, p, q);
            const double2 c = cs[g & 1][k];
            const double a = Y[row][p], b = Y[row][q];
            Y[row][p] = c.x * a - c.y * b;
            Y[row][q] = c.y * a + c.x * b;
        }
        if (++round == N - 1) round = 0;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kJacRows * na; e += 256) {
        const int r = e / na, c = e - r * na;
        if (r0 + r < na) Yg[(long)(r0 + r) * m + c] = Y[r][c];
    }
}

// theta[t] the eigenvalues sorted descending, perm[t] the column of Y of each and ylast[t]
// that column's last component
__global__ void k_ritz(const double *__restrict__ M, const double *__restrict__ Y, const int *__restrict__ nlock,
                       int m, double *__restrict__ theta, int *__restrict__ perm, double *__restrict__ ylast)
{
    __shared__ double d[160];
    const int t = blockIdx.x, na = m - nlock[t], N = na + (na & 1);
    for (int i = threadIdx.x; i < na; i += blockDim.x) d[i] = M[(long)t * m * m + fold(i, i, N)];
    __syncthreads();
    for (int i = threadIdx.x; i < na; i += blockDim.x) {
        const double di = d[i];
        int rank = 0;
        for (int k = 0; k < na; k++) rank += (d[k] > di) || (d[k] == di && k < i);
        theta[(long)t * m + rank] = di;
        perm[(long)t * m + rank] = i;
        ylast[(long)t * m + rank] = Y[((long)t * m + (na - 1)) * m + i];
    }
}

// Qtmp[t][c] = sum_{a < na} Q[t][nlock + a] Y[t][a][ycol[t][c]], c < ncols[t]
constexpr int ROT_C = 16;
__global__ __launch_bounds__(256) void k_rotate(const double2 *__restrict__ Q, long qslice, long n,
                                                const double *__restrict__ Y, const int *__restrict__ ycol,
                                                const int *__restrict__ nlock, const int *__restrict__ ncols, int m,
                                                double2 *__restrict__ Qt, long tslice)
{
    int t = blockIdx.z;
    int c0 = blockIdx.y * ROT_C;
    int nc = min(ROT_C, ncols[t] - c0);
    if (nc <= 0) return;
    int l = nlock[t], na = m - l;
    __shared__ double yc[160][ROT_C];
    for (int idx = threadIdx.x; idx < na * ROT_C; idx += blockDim.x) {
        int a = idx / ROT_C, cc = idx % ROT_C;
        yc[a][cc] = cc < nc ? Y[((long)t * m + a) * m + ycol[(long)t * m + c0 + cc]] : 0.0;
    }
    __syncthreads();
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n) return;
    double2 acc[ROT_C];
#pragma unroll
    for (int cc = 0; cc < ROT_C; cc++) acc[cc] = make_double2(0, 0);
    const double2 *q = Q + t * qslice + (long)l * n + row;
    for (int a = 0; a < na; a++) {
        double2 v = q[(long)a * n];
#pragma unroll
        for (int cc = 0; cc < ROT_C; cc++) {
            acc[cc].x += v.x * yc[a][cc];
            acc[cc].y += v.y * yc[a][cc];
        }
    }
    for (int cc = 0; cc < nc; cc++) Qt[t * tslice + (long)(c0 + cc) * n + row] = acc[cc];
}

// Q[t][nlock_old + c] = Qtmp[t][c] for c < ncols[t];  Q[t][rtot] = Q[t][m] (residual)
__global__ __launch_bounds__(256) void k_copyback(double2 *__restrict__ Q, long qslice, long n,
                                                  const double2 *__restrict__ Qt, long tslice,
                                                  const int *__restrict__ nlock_old, const int *__restrict__ ncols,
                                                  int m, int rtot)
{
    int t = blockIdx.y;
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= n) return;
    int l = nlock_old[t];
    for (int c = 0; c < ncols[t]; c++) Q[t * qslice + (long)(l + c) * n + row] = Qt[t * tslice + (long)c * n + row];
    Q[t * qslice + (long)rtot * n + row] = Q[t * qslice + (long)m * n + row];
}

// T[t] = 0 except T[p][p] = diag[t][p] for p in [lo[t], hi)
__global__ void k_set_T(double *__restrict__ T, const double *__restrict__ diag, const int *__restrict__ lo, int hi,
                        int m)
{
    int t = blockIdx.x;
    for (int idx = threadIdx.x; idx < m * m; idx += blockDim.x) {
        int i = idx / m, k = idx % m;
        double v = 0;
        if (i == k && i >= lo[t] && i < hi) v = diag[(long)t * m + i];
        T[(long)t * m * m + idx] = v;
    }
}

// per-slice <a_t, b_t> partials (a, b with their own slice strides)
__global__ __launch_bounds__(256) void k_dot_slices(const double2 *__restrict__ a, long as, const double2 *__restrict__ b,
                                                    long bs, long n, double *__restrict__ part)
{
    int t = blockIdx.y;
    __shared__ double r0[256], r1[256];
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    double re = 0, im = 0;
    if (row < n) {
        double2 u = a[t * as + row], v = b[t * bs + row];
        re = u.x * v.x + u.y * v.y;
        im = u.x * v.y - u.y * v.x;
    }
    r0[threadIdx.x] = re;
    r1[threadIdx.x] = im;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            r0[threadIdx.x] += r0[threadIdx.x + s];
            r1[threadIdx.x] += r1[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[((long)t * gridDim.x + blockIdx.x) * 2] = r0[0];
        part[((long)t * gridDim.x + blockIdx.x) * 2 + 1] = r1[0];
    }
}

// y = y + lam_t q (per slice), partial |y|^2
__global__ __launch_bounds__(256) void k_resid_slices(double2 *__restrict__ y, long n, const double2 *__restrict__ q,
                                                      long qs, const double *__restrict__ lam, double *__restrict__ part)
{
    int t = blockIdx.y;
    __shared__ double red[256];
    long row = (long)blockIdx.x * blockDim.x + threadIdx.x;
    double acc = 0;
    if (row < n) {
        double2 v = cadd(y[t * n + row], cscale(q[t * qs + row], lam[t]));
        acc = cnorm2(v);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(long)t * gridDim.x + blockIdx.x] = red[0];
}

// evecs[t][p] = phase * Q[t][src[t][p]] with the phase convention; one block per (p, t)
__global__ __launch_bounds__(256) void k_phase_out(const double2 *__restrict__ Q, long qslice, long n,
                                                   const int *__restrict__ src, int nv, double2 *__restrict__ out)
{
    int p = blockIdx.x, t = blockIdx.y;
    const double2 *v = Q + t * qslice + (long)src[t * nv + p] * n;
    __shared__ double red[256];
    __shared__ long ired[256];
    double mx = 0;
    for (long r = threadIdx.x; r < n; r += blockDim.x) mx = fmax(mx, cnorm2(v[r]));
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    double thr = 0.01 * red[0];  // |v_i| >= 0.1 max|v|  <=>  |v_i|^2 >= 0.01 max|v|^2
    long first = n;
    for (long r = threadIdx.x; r < n; r += blockDim.x)
        if (cnorm2(v[r]) >= thr) {
            first = r;
            break;
        }
    ired[threadIdx.x] = first;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) ired[threadIdx.x] = min(ired[threadIdx.x], ired[threadIdx.x + s]);
        __syncthreads();
    }
    double2 vi = v[ired[0]];
    double a = sqrt(cnorm2(vi));
    double2 ph = make_double2(vi.x / a, -vi.y / a);
    double2 *o = out + ((long)t * nv + p) * n;
    for (long r = threadIdx.x; r < n; r += blockDim.x) {
        double2 z = cmul(v[r], ph);
        if (r == ired[0]) z = make_double2(a, 0.0);
        o[r] = z;
    }
}

struct Bufs {
    double2 *Q, *Qt, *w, *w0, *w1, *coef;
    double *T, *M, *Y, *theta, *ylast, *diag, *nb, *nrm, *alpha, *npart, *beta, *lam, *dpart;
    int *flags, *nsw, *nlock, *nlock_old, *ncols, *ycol, *perm, *src;
};

}  // namespace

// scratch of laph_eigvecs (the buffers below, in the same order)
size_t eig_scratch_bytes(const Geom &g, int m, int nv)
{
    const size_t nt = g.nt, n = 3 * g.V3, V = g.V;
    const size_t rb = (n + 255) / 256, ps = m + 1;
    size_t s = 0;
    for (size_t b : {V * 36 * 16, V * 36 * 16 /* stout.tmp */, 27 * V * 16, nt * (m + 1) * n * 16, nt * m * n * 16,
                     nt * n * 16, nt * n * 16, nt * n * 16, nt * ps * 16, nt * m * m * 8, nt * m * m * 8, nt * m * m * 8, nt * m * 8, nt * m * 8, nt * m * 8, nt * 8, nt * 8, nt * 8, nt * 8,
                     nt * rb * 8, nt * 8, nt * 8, nt * rb * 16, nt * 4, nt * 4, nt * 4, nt * 4, nt * 4, nt * m * 4,
                     nt * m * 4, nt * (size_t)nv * 4})
        s += ws_align(b);
    return s;
}

extern "C" int laph_eigvecs(laph_ctx_t c, const double *U, const laph_stout *stout, const laph_lanczos *lz, int nv,
                            double *evals, double *evecs, laph_eig_stats *stats)
{
    LAPH_API_BEGIN(c)
    g_current_ctx = c;
    LAPH_CHECK(U && stout && lz && evals && evecs && nv > 0, LAPH_EINVAL, "bad arguments");
    const int nt = c->g.nt;
    const long n = 3 * c->g.V3;
    const int m = lz->krylov_dim;
    LAPH_CHECK(m <= 160 && m > nv + 12 && m <= n, LAPH_EINVAL, "krylov_dim must satisfy nv + 12 < m <= min(160, 3 Ns^3)");
    LAPH_CHECK(lz->cheb_order >= 1 && lz->lambda_L > lz->lambda_C && lz->tol > 0 && lz->max_restarts >= 0,
               LAPH_EINVAL, "bad Lanczos parameters");
    const int rtot = std::min(nv + (m - nv) / 2, m - 12);
    hipStream_t st = c->stream;

    // smeared links (SoA) for the Laplacian
    double *Us = (double *)ctx_named(c, "eig.Us", (size_t)c->g.V * 36 * 16);
    stout_smear_device(c, U, stout->rho, stout->nsteps, Us);
    double2 *us = (double2 *)ctx_named(c, "lap.us", (size_t)27 * c->g.V * 16);
    smeared_links_to_soa(c, Us, us);

    const long qslice = (long)(m + 1) * n;
    const int pstride = m + 1;
    const unsigned rb = nblocks_for(n, 256);
    Bufs b;
    b.Q = (double2 *)ctx_named(c, "eig.Q", (size_t)nt * qslice * 16);
    b.Qt = (double2 *)ctx_named(c, "eig.Qt", (size_t)nt * m * n * 16);
    b.w = (double2 *)ctx_named(c, "eig.w", (size_t)nt * n * 16);
    b.w0 = (double2 *)ctx_named(c, "eig.w0", (size_t)nt * n * 16);
    b.w1 = (double2 *)ctx_named(c, "eig.w1", (size_t)nt * n * 16);
    b.coef = (double2 *)ctx_named(c, "eig.coef", (size_t)nt * pstride * 16);
    b.T = (double *)ctx_named(c, "eig.T", (size_t)nt * m * m * 8);
    b.M = (double *)ctx_named(c, "eig.M", (size_t)nt * m * m * 8);
    b.Y = (double *)ctx_named(c, "eig.Y", (size_t)nt * m * m * 8);
    b.theta = (double *)ctx_named(c, "eig.theta", (size_t)nt * m * 8);
    b.ylast = (double *)ctx_named(c, "eig.ylast", (size_t)nt * m * 8);
    b.diag = (double *)ctx_named(c, "eig.diag", (size_t)nt * m * 8);
    b.nb = (double *)ctx_named(c, "eig.nb", (size_t)nt * 8);
    b.nrm = (double *)ctx_named(c, "eig.nrm", (size_t)nt * 8);
    double *nb0 = (double *)ctx_named(c, "eig.nb0", (size_t)nt * 8);
    b.alpha = (double *)ctx_named(c, "eig.alpha", (size_t)nt * 8);
    b.npart = (double *)ctx_named(c, "eig.npart", (size_t)nt * rb * 8);
    b.beta = (double *)ctx_named(c, "eig.beta", (size_t)nt * 8);
    b.lam = (double *)ctx_named(c, "eig.lam", (size_t)nt * 8);
    b.dpart = (double *)ctx_named(c, "eig.dpart", (size_t)nt * rb * 16);
    b.flags = (int *)ctx_named(c, "eig.flags", (size_t)nt * 4);
    b.nsw = (int *)ctx_named(c, "eig.nsw", (size_t)nt * 4);
    b.nlock = (int *)ctx_named(c, "eig.nlock", (size_t)nt * 4);
    b.nlock_old = (int *)ctx_named(c, "eig.nlock_old", (size_t)nt * 4);
    b.ncols = (int *)ctx_named(c, "eig.ncols", (size_t)nt * 4);
    b.ycol = (int *)ctx_named(c, "eig.ycol", (size_t)nt * m * 4);
    b.perm = (int *)ctx_named(c, "eig.perm", (size_t)nt * m * 4);
    b.src = (int *)ctx_named(c, "eig.src", (size_t)nt * nv * 4);

    std::vector<int> h_nlock(nt, 0), h_ncols(nt, 0), h_ycol((size_t)nt * m, 0), h_src((size_t)nt * nv);
    std::vector<double> h_theta((size_t)nt * m), h_ylast((size_t)nt * m), h_beta(nt), h_diag((size_t)nt * m, 0.0);
    std::vector<int> h_perm((size_t)nt * m), h_done(nt);
    // LDS of k_jacobi_sweeps: the folded matrix and one round's rotations
    const int jn = m + (m & 1);
    const size_t jac_lds = sizeof(double) * ((size_t)(jn / 2) * (jn + 1) + 1) + sizeof(double2) * (jn / 2);
    if (jac_lds > 64 * 1024)
        LAPH_HIP(hipFuncSetAttribute((const void *)k_jacobi_sweeps, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)jac_lds));
    std::vector<double> Anorm(nt, 0.0);
    LAPH_HIP(hipMemcpyAsync(b.nlock, h_nlock.data(), nt * 4, hipMemcpyHostToDevice, st));
    LAPH_HIP(hipMemsetAsync(b.T, 0, (size_t)nt * m * m * 8, st));

    dim3 g2(rb, nt);
    // start vector: Philox draws, normalised
    hipLaunchKernelGGL(k_random, g2, dim3(256), 0, st, b.Q, qslice, n, lz->seed);
    hipLaunchKernelGGL(k_norm_slices, g2, dim3(256), 0, st, (const double2 *)b.Q, qslice, n, b.npart);
    hipLaunchKernelGGL(k_norm_fin, dim3(nt), dim3(256), 0, st, (const double *)b.npart, (int)rb, b.nrm);
    hipLaunchKernelGGL(k_scale, g2, dim3(256), 0, st, b.Q, qslice, n, (const double *)b.nrm);
    LAPH_HIP(hipGetLastError());

    // block sums of a step, in the buffer of k_rotate (free here; far larger: its m n double2
    // per slice against nb (m + 1) + nb + 1.5 nl, with nb and nl at most n / 32 + 1)
    const int nl = lap_blocks(c->g);
    double2 *part = b.Qt;
    // workgroups per slice: two per CU over all slices for the 20-column tiles (about 200
    // registers), four for the smaller ones
    auto gs_blocks = [&](int cnt) {
        const long tiles = (n + kGsRows - 1) / kGsRows, want = (cnt > 10 * kGsGroups ? 512 : 1024) / nt;
        return (int)std::max<long>(1, std::min(tiles, want));
    };
    // one full pass of w1 (first: from w with the local part taken off) against q_0 .. q_j
    auto gs_pass = [&](int cnt, bool first) {
        const int nb = gs_blocks(cnt);
        double *wpart = (double *)(part + (size_t)nt * nb * pstride), *lsum = wpart + (size_t)nt * nb;
        gs_columns(cnt, [&](auto nc) {
            constexpr int NC = decltype(nc)::value;
            if (first)
                hipLaunchKernelGGL((k_gs_dots<NC, true>), dim3(nb, nt), dim3(256), 0, st, (const double2 *)b.Q, qslice,
                                   n, (const double2 *)b.w, b.w1, cnt, (const double *)lsum, nl, (const double *)b.T, m,
                                   b.alpha, nb0, part, pstride, wpart);
            else
                hipLaunchKernelGGL((k_gs_dots<NC, false>), dim3(nb, nt), dim3(256), 0, st, (const double2 *)b.Q, qslice,
                                   n, (const double2 *)b.w1, b.w1, cnt, (const double *)nullptr, 0,
                                   (const double *)b.T, m, b.alpha, nb0, part, pstride, wpart);
            hipLaunchKernelGGL(k_gs_fin, dim3(nt), dim3(256), 0, st, (const double2 *)part, (const double *)wpart, nb,
                               pstride, cnt, b.coef, b.nb, (const double *)b.alpha, b.T, m, (const int *)b.nlock,
                               first ? 0 : 1);
            hipLaunchKernelGGL(k_gs_update<NC>, dim3(nb, nt), dim3(256), 0, st, (const double2 *)b.Q, qslice, n, b.w1,
                               cnt, (const double2 *)b.coef, pstride, wpart);
        });
        LAPH_HIP(hipGetLastError());
    };

    int j0 = 0, restarts = 0, matvecs = 0;
    std::vector<int> last_lold(nt, 0);
    bool converged = false;
    for (;; restarts++) {
        for (int j = j0; j < m; j++) {
            const int cnt = j + 1, nb = gs_blocks(cnt);
            double *wpart = (double *)(part + (size_t)nt * nb * pstride), *lsum = wpart + (size_t)nt * nb;
            // w = A q_j, with <q_j, w> and |w|^2
            cheb_apply(c, us, b.Q + (long)j * n, qslice, b.w, n, b.w0, b.w1, n, lz->lambda_L, lz->lambda_C,
                       lz->cheb_order, lsum);
            matvecs++;
            gs_pass(cnt, true);
            // the first vector after a restart is coupled to every kept Ritz vector, so its
            // first pass shrinks it and a second is due
            const int passes = j > 0 && j == j0 ? 2 : 1;
            if (passes == 2) gs_pass(cnt, false);
            hipLaunchKernelGGL(k_gs_check, dim3(nt), dim3(1024), 0, st, (const double2 *)b.Q, qslice, n, b.w1, cnt,
                               (const double *)wpart, nb, (const double *)b.nb, (const double *)nb0, b.T, m,
                               (const int *)b.nlock, passes,
                               lz->seed + 7919u * (uint32_t)restarts + 104729u * (uint32_t)j, b.nrm,
                               j == m - 1 ? b.beta : (double *)nullptr);
            // q_{j+1} (or the residual slot m)
            hipLaunchKernelGGL(k_gs_scale, g2, dim3(256), 0, st, (const double2 *)b.w1, n, b.Q + (long)(j + 1) * n,
                               qslice, (const double *)b.nrm);
            LAPH_HIP(hipGetLastError());
        }
        // Rayleigh-Ritz on the active block
        hipLaunchKernelGGL(k_active, dim3(nt), dim3(256), 0, st, (const double *)b.T, b.M, m, (const int *)b.nlock,
                           b.flags);
        // the rotations of a launch's sweeps go to the rotation buffer of k_rotate (free
        // here; n >= m, so at least two sweeps fit); launches continue where the last one
        // stopped and return at once on finished slices, so the host looks only after ten
        const long rstride = (long)m * n;
        const int most = (int)std::min<long>(5, rstride / ((m + (m & 1) - 1) * (long)((m + 1) / 2)));
        for (int sw = 0; sw < kJacSweeps;) {
            const int until = std::min(kJacSweeps, sw + 10);
            for (; sw < until; sw += most) {
                hipLaunchKernelGGL(k_jacobi_sweeps, dim3(nt), dim3(kJacLanes), jac_lds, st, b.M, b.Qt, rstride, m,
                                   (const int *)b.nlock, most, b.nsw, b.flags);
                hipLaunchKernelGGL(k_jacobi_vectors, dim3((m + kJacRows - 1) / kJacRows, nt), dim3(256), 0, st, b.Y,
                                   (const double2 *)b.Qt, rstride, m, (const int *)b.nlock, (const int *)b.nsw,
                                   sw == 0 ? 1 : 0);
            }
            hipLaunchKernelGGL(k_ritz, dim3(nt), dim3(256), 0, st, (const double *)b.M, (const double *)b.Y,
                               (const int *)b.nlock, m, b.theta, b.perm, b.ylast);
            LAPH_HIP(hipGetLastError());
            LAPH_HIP(hipMemcpyAsync(h_done.data(), b.flags, nt * 4, hipMemcpyDeviceToHost, st));
            LAPH_HIP(hipMemcpyAsync(h_theta.data(), b.theta, h_theta.size() * 8, hipMemcpyDeviceToHost, st));
            LAPH_HIP(hipMemcpyAsync(h_ylast.data(), b.ylast, h_ylast.size() * 8, hipMemcpyDeviceToHost, st));
            LAPH_HIP(hipMemcpyAsync(h_perm.data(), b.perm, h_perm.size() * 4, hipMemcpyDeviceToHost, st));
            LAPH_HIP(hipStreamSynchronize(st));
            if (std::all_of(h_done.begin(), h_done.end(), [](int d) { return d != 0; })) break;
        }
        LAPH_HIP(hipMemcpyAsync(h_beta.data(), b.beta, nt * 8, hipMemcpyDeviceToHost, st));
        LAPH_HIP(hipStreamSynchronize(st));
        // lock / keep decisions per slice
        std::vector<int> nlock_new(nt);
        last_lold = h_nlock;
        bool all_done = true;
        for (int t = 0; t < nt; t++) {
            int l = h_nlock[t], na = m - l;
            const double *th = &h_theta[(size_t)t * m];
            const double *yl = &h_ylast[(size_t)t * m];
            for (int i = 0; i < na; i++) Anorm[t] = std::max(Anorm[t], std::fabs(th[i]));
            int want = nv - l;
            std::vector<int> lock, keep;
            std::vector<char> used(na, 0);
            for (int i = 0; i < want && i < na; i++) {
                double res = std::fabs(h_beta[t] * yl[i]);
                if (res < lz->tol * Anorm[t]) {
                    lock.push_back(i);
                    used[i] = 1;
                }
            }
            int ln = l + (int)lock.size();
            int nkeep = rtot - ln;
            for (int i = 0; i < na && (int)keep.size() < nkeep; i++)
                if (!used[i]) keep.push_back(i);
            h_ncols[t] = (int)(lock.size() + keep.size());
            int cc = 0;
            for (int i : lock) h_ycol[(size_t)t * m + cc++] = h_perm[(size_t)t * m + i];
            for (int i : keep) h_ycol[(size_t)t * m + cc++] = h_perm[(size_t)t * m + i];
            for (int k = 0; k < (int)keep.size(); k++) h_diag[(size_t)t * m + ln + k] = th[keep[k]];
            nlock_new[t] = ln;
            if (ln < nv) all_done = false;
        }
        bool stop = all_done || restarts >= lz->max_restarts;
        converged = all_done;
        // rotate the active block onto the selected Ritz vectors
        LAPH_HIP(hipMemcpyAsync(b.nlock_old, h_nlock.data(), nt * 4, hipMemcpyHostToDevice, st));
        LAPH_HIP(hipMemcpyAsync(b.ncols, h_ncols.data(), nt * 4, hipMemcpyHostToDevice, st));
        LAPH_HIP(hipMemcpyAsync(b.ycol, h_ycol.data(), h_ycol.size() * 4, hipMemcpyHostToDevice, st));
        int maxc = *std::max_element(h_ncols.begin(), h_ncols.end());
        hipLaunchKernelGGL(k_rotate, dim3(rb, (maxc + ROT_C - 1) / ROT_C, nt), dim3(256), 0, st, (const double2 *)b.Q,
                           qslice, n, (const double *)b.Y, (const int *)b.ycol, (const int *)b.nlock_old,
                           (const int *)b.ncols, m, b.Qt, (long)m * n);
        hipLaunchKernelGGL(k_copyback, g2, dim3(256), 0, st, b.Q, qslice, n, (const double2 *)b.Qt, (long)m * n,
                           (const int *)b.nlock_old, (const int *)b.ncols, m, rtot);
        LAPH_HIP(hipGetLastError());
        h_nlock = nlock_new;
        LAPH_HIP(hipMemcpyAsync(b.nlock, h_nlock.data(), nt * 4, hipMemcpyHostToDevice, st));
        if (stop) break;
        LAPH_HIP(hipMemcpyAsync(b.diag, h_diag.data(), h_diag.size() * 8, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_set_T, dim3(nt), dim3(256), 0, st, b.T, (const double *)b.diag, (const int *)b.nlock,
                           rtot, m);
        LAPH_HIP(hipGetLastError());
        j0 = rtot;
    }

    // Rayleigh quotients on -Lap and residuals for the first nv basis vectors
    std::vector<double> lam((size_t)nt * nv), res((size_t)nt * nv);
    std::vector<double> hp((size_t)nt * rb * 2);
    for (int p = 0; p < nv; p++) {
        const double2 *q = b.Q + (long)p * n;
        lap_fused(c, us, q, qslice, nullptr, 0, b.w, n, 1.0, 0.0, 0.0);
        hipLaunchKernelGGL(k_dot_slices, g2, dim3(256), 0, st, q, qslice, (const double2 *)b.w, n, n, b.dpart);
        LAPH_HIP(hipMemcpyAsync(hp.data(), b.dpart, (size_t)nt * rb * 16, hipMemcpyDeviceToHost, st));
        LAPH_HIP(hipStreamSynchronize(st));
        std::vector<double> lt(nt);
        for (int t = 0; t < nt; t++) {
            double s = 0;
            for (unsigned k = 0; k < rb; k++) s += hp[((size_t)t * rb + k) * 2];
            lt[t] = -s;  // <q, Lap q> = -lambda
            lam[(size_t)t * nv + p] = -s;
        }
        LAPH_HIP(hipMemcpyAsync(b.lam, lt.data(), nt * 8, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_resid_slices, g2, dim3(256), 0, st, b.w, n, q, qslice, (const double *)b.lam, b.npart);
        LAPH_HIP(hipMemcpyAsync(hp.data(), b.npart, (size_t)nt * rb * 8, hipMemcpyDeviceToHost, st));
        LAPH_HIP(hipStreamSynchronize(st));
        for (int t = 0; t < nt; t++) {
            double s = 0;
            for (unsigned k = 0; k < rb; k++) s += hp[(size_t)t * rb + k];
            res[(size_t)t * nv + p] = std::sqrt(s);
        }
    }
    // ascending order per slice, phase convention, canonical output
    double maxres = 0;
    for (int t = 0; t < nt; t++) {
        std::vector<int> idx(nv);
        std::iota(idx.begin(), idx.end(), 0);
        std::stable_sort(idx.begin(), idx.end(),
                         [&](int a, int bb) { return lam[(size_t)t * nv + a] < lam[(size_t)t * nv + bb]; });
        for (int p = 0; p < nv; p++) {
            h_src[(size_t)t * nv + p] = idx[p];
            evals[(size_t)t * nv + p] = lam[(size_t)t * nv + idx[p]];
            maxres = std::max(maxres, res[(size_t)t * nv + idx[p]]);
        }
    }
    LAPH_HIP(hipMemcpyAsync(b.src, h_src.data(), h_src.size() * 4, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_phase_out, dim3(nv, nt), dim3(256), 0, st, (const double2 *)b.Q, qslice, n,
                       (const int *)b.src, nv, (double2 *)evecs);
    LAPH_HIP(hipGetLastError());
    if (stats) {
        stats->restarts = restarts;
        stats->matvecs = matvecs;
        stats->max_residual = maxres;
        // orthonormality of the output: max |<v_a, v_p> - delta_ap| over slices, from the Gram
        // matrices (in the buffer of k_rotate, whose 3 m V3 double2 per slice they fit with the
        // phase: V3 / 64 pieces of nv nv < 147 m at most)
        double2 *gram = b.Qt + c->g.V3;
        const int parts = gram_parts(c->g.V3);
        const unsigned gb = std::min(rb, 16u);  // (npart holds rb values a slice)
        overlap_slices(c, (const double2 *)evecs, nv, (const double2 *)evecs, nv, 0, 0, 0, b.Qt, gram, parts);
        hipLaunchKernelGGL(k_gram_dev, dim3(gb, nt), dim3(256), 0, st, (const double2 *)gram, nv, parts, b.npart);
        LAPH_HIP(hipGetLastError());
        std::vector<double> dev((size_t)nt * gb);
        LAPH_HIP(hipMemcpyAsync(dev.data(), b.npart, dev.size() * 8, hipMemcpyDeviceToHost, st));
        LAPH_HIP(hipStreamSynchronize(st));
        const double mo = *std::max_element(dev.begin(), dev.end());
        stats->max_orth = mo;
        // gap estimate: the first Ritz value of A below the wanted ones, mapped back to -Lap
        double gap = 1e300;
        double cc = 2.0 / (lz->lambda_L - lz->lambda_C);
        for (int t = 0; t < nt; t++) {
            double th = h_theta[(size_t)t * m + (nv - last_lold[t])];
            double lam_next = lz->lambda_C;
            if (th > 1.0) lam_next = lz->lambda_C - (std::cosh(std::acosh(th) / lz->cheb_order) - 1.0) / cc;
            gap = std::min(gap, lam_next - evals[(size_t)t * nv + nv - 1]);
        }
        stats->min_gap = gap;
    }
    LAPH_HIP(hipStreamSynchronize(st));
    if (!converged) laph_fail(LAPH_EEIG, "eigensolver: not all %d pairs converged in %d restarts", nv, restarts);
    LAPH_API_END(c)
}
