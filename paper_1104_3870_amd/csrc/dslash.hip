// Even-odd anisotropic Wilson-clover hopping kernel with fused clover epilogues.
#include "spinor_io.h"

namespace {

template <typename A>
struct Spin {
    Cx<A> v[4][3];
};

template <typename A>
__device__ __forceinline__ void mat_vec(const Cx<A> (&U)[9], const Cx<A> (&h)[3], Cx<A> (&o)[3])
{
#pragma unroll
    for (int a = 0; a < 3; a++) o[a] = U[a * 3] * h[0] + U[a * 3 + 1] * h[1] + U[a * 3 + 2] * h[2];
}
template <typename A>
__device__ __forceinline__ void mat_dag_vec(const Cx<A> (&U)[9], const Cx<A> (&h)[3], Cx<A> (&o)[3])
{
#pragma unroll
    for (int a = 0; a < 3; a++) o[a] = conjmul(U[a], h[0]) + conjmul(U[3 + a], h[1]) + conjmul(U[6 + a], h[2]);
}

// Element e of a field stored as planes of Vh (links, clover) or Vh R (spinors) entries:
// plane + e.  With O32 (the launcher checks that every plane is below 4 GiB) the plane
// start stays a uniform (scalar) address and each lane adds one 32-bit byte offset, so a
// neighbour spinor costs one address register instead of twelve 64-bit pairs.
template <bool O32, typename T>
__device__ __forceinline__ const T &elem(const T *plane, long e)
{
    if constexpr (O32)
        return *(const T *)((const char *)plane + ((unsigned)e * (unsigned)sizeof(T)));
    else
        return plane[e];
}
template <bool O32, typename T>
__device__ __forceinline__ T &elem(T *plane, long e)
{
    if constexpr (O32)
        return *(T *)((char *)plane + ((unsigned)e * (unsigned)sizeof(T)));
    else
        return plane[e];
}

template <class GP, typename A, bool O32>
__device__ __forceinline__ void load_link(const typename GP::E *g, int mu, int par, long Vh, long i, Cx<A> (&U)[9])
{
    const typename GP::E *p = g + (long)(mu * 2 + par) * 9 * Vh;
#pragma unroll
    for (int k = 0; k < 9; k++) {
        const auto v = elem<O32>(p + (long)k * Vh, i);
        U[k] = {(A)v.x, (A)v.y};
    }
}

template <class SP, bool O32>
__device__ __forceinline__ void load_spinor(const typename SP::E *s, const float *nrm, long Vh, int R, long i, int r,
                                            Spin<typename SP::A> &out)
{
    Cx<typename SP::A> v[12];
    if constexpr (O32) {
        static_assert(std::is_same<SP, S64>::value, "32-bit offsets: FP64 plane layout only");
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double2 e = elem<true>(s + (long)k * Vh * R, i * R + r);
            v[k] = {e.x, e.y};
        }
    } else {
        ld_spinor12<SP, typename SP::A>(s, nrm, Vh, R, i, r, v);
    }
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int c = 0; c < 3; c++) out.v[a][c] = v[a * 3 + c];
}

template <class SP, bool O32>
__device__ __forceinline__ void store_spinor(typename SP::E *s, float *nrm, long Vh, int R, long i, int r,
                                             const Spin<typename SP::A> &in)
{
    Cx<typename SP::A> v[12];
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int c = 0; c < 3; c++) v[a * 3 + c] = in.v[a][c];
    if constexpr (O32) {
        static_assert(std::is_same<SP, S64>::value, "32-bit offsets: FP64 plane layout only");
#pragma unroll
        for (int k = 0; k < 12; k++) elem<true>(s + (long)k * Vh * R, i * R + r) = make_double2(v[k].re, v[k].im);
    } else {
        st_spinor12<SP, typename SP::A>(s, nrm, Vh, R, i, r, v);
    }
}

// packed Hermitian 6x6 block times a 6-vector
template <class CP, typename A, bool O32 = false>
__device__ __forceinline__ void herm6(const typename CP::E *cl, long Vh, long i, const Cx<A> (&v)[6], Cx<A> (&o)[6])
{
    A d[6];
#pragma unroll
    for (int k = 0; k < 6; k++) d[k] = (A)elem<O32>(cl + (long)k * Vh, i);
#pragma unroll
    for (int k = 0; k < 6; k++) o[k] = d[k] * v[k];
    int e = 6;
#pragma unroll
    for (int r = 1; r < 6; r++)
#pragma unroll
        for (int c = 0; c < r; c++) {
            Cx<A> L = {(A)elem<O32>(cl + (long)e * Vh, i), (A)elem<O32>(cl + (long)(e + 1) * Vh, i)};
            e += 2;
            o[r] = o[r] + L * v[c];
            o[c] = o[c] + conjmul(L, v[r]);
        }
}

template <class CP, typename A, bool O32 = false>
__device__ __forceinline__ void clover_mul(const typename CP::E *cl, long Vh, long i, const Spin<A> &in, Spin<A> &out)
{
#pragma unroll
    for (int blk = 0; blk < 2; blk++) {
        Cx<A> v[6], o[6];
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
            for (int c = 0; c < 3; c++) v[s * 3 + c] = in.v[blk * 2 + s][c];
        herm6<CP, A, O32>(cl + (long)blk * 36 * Vh, Vh, i, v, o);
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
            for (int c = 0; c < 3; c++) out.v[blk * 2 + s][c] = o[s * 3 + c];
    }
}

template <typename A>
__device__ __forceinline__ void acc_upper(Spin<A> &acc, const Cx<A> (&w0)[3], const Cx<A> (&w1)[3])
{
#pragma unroll
    for (int c = 0; c < 3; c++) {
        acc.v[0][c] = acc.v[0][c] + w0[c];
        acc.v[1][c] = acc.v[1][c] + w1[c];
    }
}

// Rolled FP64 hops: one loop trip per direction d = 2 mu + (backward), the spin structure
// of (1 -/+ gamma_mu) taken from per-direction unit coefficients, so that only one
// direction's neighbour and link are live at a time (150 instead of ~290 registers: three
// waves per SIMD instead of one for this latency-bound kernel).
// h0 = w s0 + a0 s_p0, h1 = w s1 + a1 s_p1 (p0, p1) = (3, 2) for mu < 2, else (2, 3);
// acc0 += o0, acc1 += o1, acc2 += b2 o_q2, acc3 += b3 o_q3 with (q2, q3) = (1, 0) for
// mu < 2, else (0, 1); forward units below (the gamma matrices of the chiral basis),
// backward hops negate them and take U_mu(x - mu)^dag.
struct HopCoef {
    double a0r, a0i, a1r, a1i, b2r, b2i, b3r, b3i;
};
__host__ __device__ constexpr HopCoef hop_coef(int mu)
{
    return mu == 0   ? HopCoef{0, 1, 0, 1, 0, -1, 0, -1}
           : mu == 1 ? HopCoef{1, 0, -1, 0, -1, 0, 1, 0}
           : mu == 2 ? HopCoef{0, 1, 0, -1, 0, -1, 0, 1}
                     : HopCoef{-1, 0, -1, 0, -1, 0, -1, 0};
}
__device__ __forceinline__ Cx<double> unit_mul(double ur, double ui, Cx<double> z)
{
    return {ur * z.re - ui * z.im, ur * z.im + ui * z.re};
}

// checkerboard index of the neighbour in direction d
__device__ __forceinline__ long neighbour(const DslashArgs &P, int d, int x, int y, int z, int t)
{
    const int mu = d >> 1, st = d & 1 ? -1 : 1, ns = P.ns;
    auto wrap = [](int a, int m) { return a < 0 ? a + m : a >= m ? a - m : a; };
    if (mu == 0) x = wrap(x + st, ns);
    if (mu == 1) y = wrap(y + st, ns);
    if (mu == 2) z = wrap(z + st, ns);
    if (mu == 3) t = wrap(t + st, P.nt);
    return lex_index(x, y, z, t, ns) >> 1;
}

// hop(o0, o1, q, sb, sw) gets the link of direction d times the two colour vectors of the
// neighbour's projected half spinor, hop weight and boundary factor included, and what the
// lower components take of them: acc2 += sb b2 (sw ? o1 : o0), acc3 += sb b3 (sw ? o0 : o1)
// kStage: staged are the nine link elements of this site and direction in LDS, as the product
// takes them (else they are read from the field)
template <bool O32, bool kStage, class F>
__device__ __forceinline__ void hop_dir(const DslashArgs &P, int d, long i, int r, int x, int y, int z, int t,
                                        const double2 *staged, F hop)
{
    // (a table of the function's own: a shared one costs the rolled kernel 36 registers)
    constexpr HopCoef kc[4] = {hop_coef(0), hop_coef(1), hop_coef(2), hop_coef(3)};
    const int R = P.R, par = P.par;
    const long Vh = P.Vh;
    const double2 *in = (const double2 *)P.in;
    const double2 *g = (const double2 *)P.gauge;
    const int mu = d >> 1;
    const bool fwd = !(d & 1);
    double w = mu == 3 ? P.wt : P.ws;
    if (mu == 3 && (fwd ? t + 1 == P.nt : t == 0)) w *= P.bct;
    const long nb = neighbour(P, d, x, y, z, t);
    Spin<double> s;
    load_spinor<S64, O32>(in, nullptr, Vh, R, nb, r, s);
    // U_mu(x), or for the backward hop U_mu(x - mu)^dag: planes read transposed, conjugated
    const double2 *gp = g + (long)(mu * 2 + (fwd ? par : par ^ 1)) * 9 * Vh;
    const long li = fwd ? i : nb;
    const double cj = fwd ? 1.0 : -1.0;
    Cx<double> U[9];
    if constexpr (!kStage) {
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const double2 v = elem<O32>(gp + (long)(fwd ? k : (k % 3) * 3 + k / 3) * Vh, li);
            U[k] = {v.x, cj * v.y};
        }
    }
    const HopCoef &q = kc[mu];
    const double sa = fwd ? w : -w, sb = fwd ? 1.0 : -1.0;
    const bool sw = mu < 2;
    Cx<double> h0[3], h1[3], o0[3], o1[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        h0[c] = w * s.v[0][c] + unit_mul(sa * q.a0r, sa * q.a0i, sw ? s.v[3][c] : s.v[2][c]);
        h1[c] = w * s.v[1][c] + unit_mul(sa * q.a1r, sa * q.a1i, sw ? s.v[2][c] : s.v[3][c]);
    }
    if constexpr (kStage) {
        // (not before the spinor is used up: the registers of both cost a wave per SIMD)
#pragma unroll
        for (int k = 0; k < 9; k++) U[k] = {staged[k].x, staged[k].y};
    }
    mat_vec(U, h0, o0);
    mat_vec(U, h1, o1);
    hop(o0, o1, q, sb, sw);
}

template <bool O32, bool kStage>
__device__ __forceinline__ void hop_rolled(const DslashArgs &P, long i, int r, int x, int y, int z, int t,
                                           const double2 *staged, Spin<double> &acc)
{
#pragma unroll 1
    for (int d = 0; d < 8; d++)
        hop_dir<O32, kStage>(P, d, i, r, x, y, z, t, kStage ? staged + 9 * d : nullptr,
                     [&](const Cx<double> (&o0)[3], const Cx<double> (&o1)[3], const HopCoef &q, double sb, bool sw) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                acc.v[0][c] = acc.v[0][c] + o0[c];
                acc.v[1][c] = acc.v[1][c] + o1[c];
                acc.v[2][c] = acc.v[2][c] + unit_mul(sb * q.b2r, sb * q.b2i, sw ? o1[c] : o0[c]);
                acc.v[3][c] = acc.v[3][c] + unit_mul(sb * q.b3r, sb * q.b3i, sw ? o0[c] : o1[c]);
            }
        });
}

// checkerboard index and coordinates of position pos of the tiled site walk: tiles of
// Ns x by x bz sites (x halved by the parity), one after the other, each visited slice by
// slice through all Nt slices; the time neighbours of a tile slice are the tile slices just
// before and after it in the walk, so that with many right-hand sides per site they are
// still in L2 (in checkerboard order they are Ns^3 / 2 sites away)
__device__ __forceinline__ long walk_coords(unsigned pos, int ns, int nt, int par, int by, int bz, int &x, int &y,
                                            int &z, int &t)
{
    const unsigned nsh = (unsigned)ns >> 1, A = nsh * by * bz;
    const unsigned q = pos / A, loc = pos - q * A;
    const unsigned tile = q / (unsigned)nt;
    t = (int)(q - tile * nt);
    const unsigned q1 = loc / nsh, xh = loc - q1 * nsh;
    const unsigned zz = q1 / (unsigned)by, yy = q1 - zz * by;
    const unsigned nty = (unsigned)ns / by, tz = tile / nty, ty = tile - tz * nty;
    y = (int)(ty * by + yy);
    z = (int)(tz * bz + zz);
    x = 2 * (int)xh + ((y + z + t + par) & 1);
    return (long)xh + (long)nsh * (y + (long)ns * (z + (long)ns * t));
}

// q += (Re <y, v>, Im <y, v>, |v|^2) of one component
__device__ __forceinline__ void dot_add(Cx<double> y, Cx<double> v, double (&q)[3])
{
    q[0] += y.re * v.re + y.im * v.im;
    q[1] += y.re * v.im - y.im * v.re;
    q[2] += v.re * v.re + v.im * v.im;
}
// sums over the lanes of a wave that hold the same right-hand side (lane mod R), in every lane
__device__ __forceinline__ void wave_sum_rhs(double (&q)[3], int R)
{
    for (int off = 32; off >= R; off >>= 1)
#pragma unroll
        for (int k = 0; k < 3; k++) q[k] += __shfl_xor(q[k], off, 64);
}

// kStage (R = 8, 16 or 32 right-hand sides: a block holds 256 / R whole sites): the block's
// links and clover elements go through LDS.  Read per lane they are half of the bytes the
// vector cache returns, although all R lanes of a site read the same ones, and they push the
// neighbours' records out of it.  24^3 x 32, R = 32: 1.50 -> 1.16 ms, 1.13 with the walk's
// tiles below, now bound by the traffic behind L2 (9.8 -> 8.2 GB, 7.2 TB/s); 16^3 x 32:
// 458 -> 363 us; R = 16: 799 -> 610, R = 8 on 16^3 x 32: 135 -> 119 us.
template <class SP, class GP, class CP, int MODE, bool O32, bool kStage>
__global__ __launch_bounds__(256) void k_dslash(const DslashArgs P)
{
    using A = typename SP::A;
    unsigned b = xcd_block(blockIdx.x, gridDim.x);
    long tid = (long)b * blockDim.x + threadIdx.x;
    const int R = P.R;
    const long Vh = P.Vh;
    constexpr bool kDot = MODE == M_INV_AFTER_DOT;
    const bool valid = tid < Vh * R;
    if (!kDot && !kStage && !valid) return;
    if (!valid) tid = Vh * R - 1;  // (lanes past the end take part in the staging and the sums, with zeros)
    // 32-bit lane arithmetic: the launcher guarantees Vh R < 2^28
    const unsigned pos = (unsigned)tid / (unsigned)R;
    const int r = (int)((unsigned)tid - pos * (unsigned)R);
    const int ns = P.ns, nt = P.nt, par = P.par, opar = par ^ 1;
    int x, y, z, t;
    long i;
    if (P.wby) {
        i = walk_coords(pos, ns, nt, par, P.wby, P.wbz, x, y, z, t);
    } else {
        i = pos;
        cb_coords(i, par, ns, x, y, z, t);
    }
    extern __shared__ double2 stage[];  // [site][8][9] links, then [site][72] clover elements
    const double2 *staged = nullptr;
    const auto *cl = (const typename CP::E *)P.clov;
    long cl_plane = Vh, cl_site = i;
    if constexpr (kStage) {
        const int S = 256 / R, s = threadIdx.x & (S - 1), e0 = threadIdx.x / S;  // (sites fastest: coalesced)
        const unsigned sp = min(b * (unsigned)S + s, (unsigned)Vh - 1);
        int sx, sy, sz, st;
        long si;
        if (P.wby) {
            si = walk_coords(sp, ns, nt, par, P.wby, P.wbz, sx, sy, sz, st);
        } else {
            si = sp;
            cb_coords(si, par, ns, sx, sy, sz, st);
        }
        double *clov = (double *)(stage + 72 * S);
        const double2 *g = (const double2 *)P.gauge;
#pragma unroll 3
        for (int e = e0; e < 72; e += R) {
            const int d = e / 9, k = e - 9 * d;
            const bool back = d & 1;
            const long li = back ? neighbour(P, d, sx, sy, sz, st) : si;
            const double2 v = elem<O32>(g + ((long)((d >> 1) * 2 + (back ? opar : par)) * 9 +
                                             (back ? (k % 3) * 3 + k / 3 : k)) * Vh, li);
            stage[72 * s + e] = make_double2(v.x, back ? -v.y : v.y);
            if constexpr (MODE != M_PLAIN) clov[72 * s + e] = elem<O32>((const double *)P.clov + (long)e * Vh, si);
        }
        __syncthreads();
        staged = stage + 72 * (threadIdx.x / R);
        cl = (const typename CP::E *)clov + 72 * (threadIdx.x / R);
        cl_plane = 1;
        cl_site = 0;
    }

    Spin<A> acc;
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int c = 0; c < 3; c++) acc.v[a][c] = {(A)0, (A)0};

    hop_rolled<O32, kStage>(P, i, r, x, y, z, t, staged, acc);

    if (P.g5d) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            acc.v[2][c] = cneg(acc.v[2][c]);
            acc.v[3][c] = cneg(acc.v[3][c]);
        }
    }

    const A ca = (A)P.a, cc = (A)P.c;
    Spin<A> res;
    if constexpr (MODE == M_PLAIN) {
#pragma unroll
        for (int a = 0; a < 4; a++)
#pragma unroll
            for (int c = 0; c < 3; c++) res.v[a][c] = cc * acc.v[a][c];
        if (P.x) {
            Spin<A> xv;
            load_spinor<SP, O32>((const typename SP::E *)P.x, P.x_nrm, Vh, R, i, r, xv);
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 3; c++) res.v[a][c] = res.v[a][c] + ca * xv.v[a][c];
        }
    } else if constexpr (MODE == M_INV_AFTER || kDot) {
        Spin<A> m;
        clover_mul<CP, A, O32>(cl, cl_plane, cl_site, acc, m);
#pragma unroll
        for (int a = 0; a < 4; a++)
#pragma unroll
            for (int c = 0; c < 3; c++) res.v[a][c] = cc * m.v[a][c];
        if (P.x) {
            Spin<A> xv;
            load_spinor<SP, O32>((const typename SP::E *)P.x, P.x_nrm, Vh, R, i, r, xv);
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 3; c++) res.v[a][c] = res.v[a][c] + ca * xv.v[a][c];
        }
    } else if constexpr (MODE == M_INV_OF_SUM) {
        Spin<A> xv, sum;
        load_spinor<SP, O32>((const typename SP::E *)P.x, P.x_nrm, Vh, R, i, r, xv);
#pragma unroll
        for (int a = 0; a < 4; a++)
#pragma unroll
            for (int c = 0; c < 3; c++) sum.v[a][c] = ca * xv.v[a][c] + cc * acc.v[a][c];
        clover_mul<CP, A, O32>(cl, cl_plane, cl_site, sum, res);
    } else {  // M_CLOV_ADD
        Spin<A> xv, m;
        load_spinor<SP, O32>((const typename SP::E *)P.x, P.x_nrm, Vh, R, i, r, xv);
        clover_mul<CP, A, O32>(cl, cl_plane, cl_site, xv, m);
#pragma unroll
        for (int a = 0; a < 4; a++)
#pragma unroll
            for (int c = 0; c < 3; c++) res.v[a][c] = m.v[a][c] + cc * acc.v[a][c];
    }
    if (valid) store_spinor<SP, O32>((typename SP::E *)P.out, P.out_nrm, Vh, R, i, r, res);
    if constexpr (kDot) {
        __shared__ double red[256 / 64][32][3];
        double q[3] = {0.0, 0.0, 0.0};
        if (valid) {
            Spin<A> y;
            load_spinor<SP, O32>((const typename SP::E *)P.dot_y, nullptr, Vh, R, i, r, y);
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 3; c++) dot_add(y.v[a][c], res.v[a][c], q);
        }
        wave_sum_rhs(q, R);
        const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
        if (lane < R)
#pragma unroll
            for (int k = 0; k < 3; k++) red[wave][lane][k] = q[k];
        __syncthreads();
        if ((int)threadIdx.x < R)
#pragma unroll
            for (int k = 0; k < 3; k++)
                P.partial[((long)blockIdx.x * R + threadIdx.x) * 3 + k] =
                    red[0][threadIdx.x][k] + red[1][threadIdx.x][k] + red[2][threadIdx.x][k] + red[3][threadIdx.x][k];
    }
}

// The FP64 hop of launches with few (site, right-hand side) pairs: the rolled kernel above
// walks eight directions one memory latency after the other, which is what bounds it while
// the chip is not full.  Here a workgroup takes 64 pairs with one wave per direction, so all
// eight neighbours are read at once; the products go through LDS, and twelve waves, one per
// spin-colour component, add them up in direction order and multiply by their row of the
// clover block, whose elements they loaded at the start.  256 sites of one parity of 4^3 x 8
// (between events): 15.6 us rolled, 9.2 us with two waves for the sums, one per chirality, and
// general integer divisions ahead of the first load, 7.9 us here.
constexpr int kSplit = 64;

// (br + i bi) z with one of the two zero and the other +-1, known at compile time
__device__ __forceinline__ Cx<double> unit_of(double br, double bi, Cx<double> z)
{
    return br != 0.0 ? Cx<double>{br * z.re, br * z.im} : Cx<double>{-bi * z.im, bi * z.re};
}

// component c of spin S of the sum over directions, from ex[direction][colour vector][pair]
template <int S>
__device__ __forceinline__ Cx<double> split_sum(const double2 (&ex)[8][6][kSplit], int c, int l)
{
    constexpr HopCoef kc[4] = {hop_coef(0), hop_coef(1), hop_coef(2), hop_coef(3)};
    Cx<double> acc = {0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const HopCoef &q = kc[e >> 1];
        const double sb = (e & 1) ? -1.0 : 1.0;
        const bool second = S == 1 || (S == 2 ? e < 4 : S == 3 && e >= 4);  // o1 or o0
        const double2 a = ex[e][(second ? 3 : 0) + c][l];
        const Cx<double> u = {a.x, a.y};
        acc = acc + (S < 2 ? u : unit_of(sb * (S == 2 ? q.b2r : q.b3r), sb * (S == 2 ? q.b2i : q.b3i), u));
    }
    return acc;
}

template <int MODE>
__global__ __launch_bounds__(12 * kSplit) void k_dslash_split(const DslashArgs P)
{
    __shared__ double2 ex[8][6][kSplit], mid[12][kSplit];
    constexpr bool kClov = MODE != M_PLAIN, kDot = MODE == M_INV_AFTER_DOT;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kSplit), l = threadIdx.x & (kSplit - 1);
    const unsigned n = (unsigned)(P.Vh * P.R), R = P.R, ns = P.ns;
    const unsigned tid = xcd_block(blockIdx.x, gridDim.x) * kSplit + l;
    const bool valid = tid < n;
    // (lanes past the end read site 0 and store nothing)
    const unsigned i = valid ? udiv(tid, R, P.m_R) : 0, r = valid ? tid - i * R : 0;
    const unsigned row = udiv(i, ns / 2, P.m_nsh), row2 = udiv(row, ns, P.m_ns), t = udiv(row2, ns, P.m_ns);
    const int y = row - row2 * ns, z = row2 - t * ns;
    const int x = 2 * (int)(i - row * (ns / 2)) + ((y + z + (int)t + P.par) & 1);
    // this wave's component, its clover row and its operands
    const int s = w / 3, ch = w / 6, k = w % 6;
    double cd = 0.0, cl[5][2];
    if constexpr (kClov) {
        const double *C = (const double *)P.clov + (long)(ch * 36) * P.Vh;
        cd = elem<true>(C + (long)k * P.Vh, i);
#pragma unroll
        for (int j = 0; j < 5; j++) {
            const int c = j < k ? j : j + 1, hi = max(k, c), lo = min(k, c), e = 6 + hi * (hi - 1) + 2 * lo;
            cl[j][0] = elem<true>(C + (long)e * P.Vh, i);
            cl[j][1] = elem<true>(C + (long)(e + 1) * P.Vh, i);
        }
    }
    const long own = (long)w * n;  // plane of this component
    Cx<double> xv = {0.0, 0.0}, yv = {0.0, 0.0};
    if (P.x) {
        const double2 e = elem<true>((const double2 *)P.x + own, i * R + r);
        xv = {e.x, e.y};
    }
    if constexpr (kDot) {
        const double2 e = elem<true>((const double2 *)P.dot_y + own, i * R + r);
        yv = {e.x, e.y};
    }
    if (w < 8)
        hop_dir<true, false>(P, w, i, r, x, y, z, t, nullptr,
                      [&](const Cx<double> (&o0)[3], const Cx<double> (&o1)[3], const HopCoef &, double, bool) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                ex[w][c][l] = make_double2(o0[c].re, o0[c].im);
                ex[w][3 + c][l] = make_double2(o1[c].re, o1[c].im);
            }
        });
    __syncthreads();
    const int c = w - 3 * s;
    Cx<double> acc = s == 0 ? split_sum<0>(ex, c, l) : s == 1 ? split_sum<1>(ex, c, l)
                   : s == 2 ? split_sum<2>(ex, c, l) : split_sum<3>(ex, c, l);
    if (P.g5d && s >= 2) acc = cneg(acc);
    const double ca = P.a, cc = P.c;
    Cx<double> m = acc;
    if constexpr (kClov) {
        if constexpr (MODE == M_INV_OF_SUM) m = ca * xv + cc * acc;
        if constexpr (MODE == M_CLOV_ADD) m = xv;
        mid[w][l] = make_double2(m.re, m.im);
        __syncthreads();
        m = cd * m;
#pragma unroll
        for (int j = 0; j < 5; j++) {
            const int o = j < k ? j : j + 1;
            const double2 v = mid[ch * 6 + o][l];
            m = m + Cx<double>{cl[j][0], j < k ? cl[j][1] : -cl[j][1]} * Cx<double>{v.x, v.y};
        }
    }
    Cx<double> res = m;
    if constexpr (MODE == M_CLOV_ADD) {
        res = m + cc * acc;
    } else if constexpr (MODE != M_INV_OF_SUM) {
        res = cc * m;
        if (P.x) res = res + ca * xv;
    }
    if (valid) elem<true>((double2 *)P.out + own, i * R + r) = make_double2(res.re, res.im);
    if constexpr (kDot) {
        double q[3] = {0.0, 0.0, 0.0};
        if (valid) dot_add(yv, res, q);
        wave_sum_rhs(q, R);
        double(*red)[32][3] = (double(*)[32][3])ex;  // (every read of ex lies before the last barrier)
        if (l < (int)R)
#pragma unroll
            for (int e = 0; e < 3; e++) red[w][l][e] = q[e];
        __syncthreads();
        if (threadIdx.x < R)
#pragma unroll
            for (int e = 0; e < 3; e++) {
                double sum = 0.0;
#pragma unroll
                for (int b = 0; b < 12; b++) sum += red[b][threadIdx.x][e];
                P.partial[((long)blockIdx.x * R + threadIdx.x) * 3 + e] = sum;
            }
    }
}

template <class SP, class CP>
__global__ __launch_bounds__(256) void k_clover_apply(const typename CP::E *__restrict__ cl,
                                                       const typename SP::E *__restrict__ x, const float *x_nrm,
                                                       typename SP::E *__restrict__ out, float *out_nrm, long Vh,
                                                       int R, int g5_in)
{
    using A = typename SP::A;
    long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (tid >= Vh * R) return;
    long i = tid / R;
    int r = (int)(tid - i * R);
    Spin<A> v, o;
    load_spinor<SP, false>(x, x_nrm, Vh, R, i, r, v);
    if (g5_in) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            v.v[2][c] = cneg(v.v[2][c]);
            v.v[3][c] = cneg(v.v[3][c]);
        }
    }
    clover_mul<CP, A>(cl, Vh, i, v, o);
    store_spinor<SP, false>(out, out_nrm, Vh, R, i, r, o);
}

}  // namespace

double dslash_bytes(long Vh, int R, int gbytes, int cbytes, int sbytes, bool has_norm, int mode, bool has_x,
                    bool y_is_x)
{
    // algorithmic bytes: 8 links, the clover block set if used, one input spinor per
    // site (neighbour re-reads are cache traffic), the output, the epilogue operand and the
    // dot epilogue's y where it is another field
    double site = 8.0 * 9 * gbytes;
    if (mode != M_PLAIN) site += 72.0 * cbytes;
    const int streams = 2 + (has_x ? 1 : 0) + (mode == M_INV_AFTER_DOT && !y_is_x ? 1 : 0);
    double per_rhs = 12.0 * sbytes * streams + (has_norm ? 4.0 * streams : 0.0);
    return (double)Vh * (site + R * per_rhs);
}

[[noreturn]] static void bad_mode(int mode) { laph_fail(LAPH_EINVAL, "no FP64 hopping kernel with epilogue mode %d", mode); }

template <class SP, class GP, class CP, bool kStage>
void launch_modes(int mode, dim3 grid, dim3 block, size_t lds, hipStream_t st, const DslashArgs &a)
{
    switch (mode) {
    case M_PLAIN: hipLaunchKernelGGL((k_dslash<SP, GP, CP, M_PLAIN, true, kStage>), grid, block, lds, st, a); return;
    case M_INV_AFTER: hipLaunchKernelGGL((k_dslash<SP, GP, CP, M_INV_AFTER, true, kStage>), grid, block, lds, st, a); return;
    case M_INV_OF_SUM: hipLaunchKernelGGL((k_dslash<SP, GP, CP, M_INV_OF_SUM, true, kStage>), grid, block, lds, st, a); return;
    case M_CLOV_ADD: hipLaunchKernelGGL((k_dslash<SP, GP, CP, M_CLOV_ADD, true, kStage>), grid, block, lds, st, a); return;
    case M_INV_AFTER_DOT:
        if constexpr (!kStage) {
            hipLaunchKernelGGL((k_dslash<SP, GP, CP, M_INV_AFTER_DOT, true, false>), grid, block, lds, st, a);
            return;
        }
    }
    bad_mode(mode);
}

// pairs up to which the split kernel is the faster one (between events, rolled against split):
// 256: 15.6 / 7.9 us, 4096: 16.6 / 9.3, 13824: 19.5 / 10.9, 32768: 20.6 / 18.9; with 65536 it is
// 2% behind, 9% with 32 right-hand sides, with 131072 (R = 32) 31.9 / 40.0 us
constexpr long kSplitMost = 32768;

void launch_split(int mode, long n, hipStream_t st, const DslashArgs &a)
{
    const dim3 grid(nblocks_for(n, kSplit)), block(12 * kSplit);
    switch (mode) {
    case M_PLAIN: hipLaunchKernelGGL(k_dslash_split<M_PLAIN>, grid, block, 0, st, a); return;
    case M_INV_AFTER: hipLaunchKernelGGL(k_dslash_split<M_INV_AFTER>, grid, block, 0, st, a); return;
    case M_INV_OF_SUM: hipLaunchKernelGGL(k_dslash_split<M_INV_OF_SUM>, grid, block, 0, st, a); return;
    case M_CLOV_ADD: hipLaunchKernelGGL(k_dslash_split<M_CLOV_ADD>, grid, block, 0, st, a); return;
    case M_INV_AFTER_DOT: hipLaunchKernelGGL(k_dslash_split<M_INV_AFTER_DOT>, grid, block, 0, st, a); return;
    }
    bad_mode(mode);
}

int dslash_dot_parts(long Vh, int R)
{
    const long n = Vh * R;
    return (int)nblocks_for(n, n <= kSplitMost ? kSplit : 256);
}

template <class SP, class GP, class CP>
void launch_dslash(laph_ctx *c, int mode, const DslashArgs &a, hipStream_t st)
{
    long n = a.Vh * a.R;
    dim3 grid(nblocks_for(n, 256)), block(256);
    hipEvent_t e0, e1;
    timing_begin(c, &e0, &e1);
    // 32-bit lane offsets: every spinor plane (Vh R entries) stays below 4 GiB (the link
    // and clover planes are smaller); callers split larger batches
    LAPH_CHECK((unsigned long long)n * sizeof(double2) < (1ull << 32), LAPH_EINVAL,
               "%d FP64 fields of %ld sites exceed the hopping kernel's 32-bit offsets", a.R, a.Vh);
    // many right-hand sides per site: a site's records span R x 192 B, so the time
    // neighbours of checkerboard order (Ns^3 / 2 sites away) fall out of L2; walk tiles
    // through time instead, the largest of which three slices stay in L2 (24^3 x 32, R = 32,
    // staged: 12 x 12 1.22, 6 x 6 1.13, 3 x 3 1.16, 2 x 2 1.28 ms; 16^3 x 32: 4 x 4 363, 2 x 2 382 us)
    DslashArgs b = a;
    b.wby = b.wbz = 0;
    if (a.R >= 8) b.wby = b.wbz = a.ns % 6 == 0 ? 6 : a.ns % 4 == 0 ? 4 : 2;
    b.m_R = umulhi_magic(a.R);  // (exact: every index is below kSplitMost)
    b.m_nsh = umulhi_magic(a.ns / 2);
    b.m_ns = umulhi_magic(a.ns);
    if (n <= kSplitMost)
        launch_split(mode, n, st, b);
    else if (mode != M_INV_AFTER_DOT && (a.R == 8 || a.R == 16 || a.R == 32))
        launch_modes<SP, GP, CP, true>(mode, grid, block, (size_t)(256 / a.R) * 72 * (sizeof(double2) + sizeof(double)),
                                       st, b);
    else
        launch_modes<SP, GP, CP, false>(mode, grid, block, 0, st, b);
    LAPH_HIP(hipGetLastError());
    if (e0)
        timing_end(c, e0, e1,
                   dslash_bytes(a.Vh, a.R, GP::bytes, CP::bytes, SP::bytes, SP::kNorm, mode, a.x != nullptr,
                                a.dot_y == a.x),
                   timing_label("dslash", SP::bytes == 16 ? "f64" : "f32", mode, a.R));
}

template <class SP, class CP>
void launch_clover_apply(laph_ctx *c, const void *clov, const void *x, const float *x_nrm, void *out, float *out_nrm,
                         long Vh, int R, int g5_in, hipStream_t st)
{
    long n = Vh * R;
    hipLaunchKernelGGL((k_clover_apply<SP, CP>), dim3(nblocks_for(n, 256)), dim3(256), 0, st,
                       (const typename CP::E *)clov, (const typename SP::E *)x, x_nrm, (typename SP::E *)out,
                       out_nrm, Vh, R, g5_in);
    LAPH_HIP(hipGetLastError());
}

template void launch_dslash<S64, G64, C64>(laph_ctx *, int, const DslashArgs &, hipStream_t);
template void launch_clover_apply<S64, C64>(laph_ctx *, const void *, const void *, const float *, void *, float *,
                                            long, int, int, hipStream_t);
