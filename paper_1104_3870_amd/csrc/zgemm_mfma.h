// Batched complex FP64 products C = A B on the FP64 matrix cores (v_mfma_f64_16x16x4f64),
// the dense contractions of the hadron functions: momentum overlaps of displaced LapH
// vectors and the baryon functions of noise fields.
//
// A workgroup of four waves computes a 64 x 64 tile of C as up to 16 tiles of 16 x 16,
// dealt to the waves in equal runs (a 48 x 64 corner costs three tiles a wave, not four).  K
// is staged through LDS KT values at a time, complex numbers whole, in two buffers: one
// barrier a stage, the next stage's global loads in flight during the products.  A complex
// product takes four real MFMAs per K step of 4: C_re += A_re B_re - A_im B_im,
// C_im += A_re B_im + A_im B_re.  Vector instructions share the FP64 pipe with the matrix
// ones (measured: they add up), so a lane's addresses are formed once and advance by a
// scalar; rows past the end read the last row (their results are not stored), values past
// the end of K are staged as zero.
//
// Lane layout of the 16 x 16 x 4 FP64 MFMA (lane l of 64): A operand A[l % 16][l / 16],
// B operand B[l / 16][l % 16], result element v of lane l at C[l / 16 + 4 v][l % 16].
#pragma once

#include <hip/hip_runtime.h>

namespace zg {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kTM = 64, kTN = 64;  // workgroup tile
constexpr int kRow = kTM + 2;      // LDS row (double2): 16-byte writes along k fall on distinct banks

// one operand of a product: rows (of A) or columns (of B) r and K index k at
// p[r * sr + k * sk], one of the strides being 1; conj: its conjugate enters; phase (may be
// null): multiplied by phase[k / 3] (KT and K multiples of 3)
struct Side {
    const double2 *p;
    long sr, sk;
    int rows;
    int conj;
    const double2 *phase;
};

// S provides: int M, N, K, tiles_m, tiles_n (64 x 64 tiles per batch), long batches;
// __device__ Side a(long batch), b(long batch); __device__ void store(long batch, int m, int n,
// double re, double im) const.
// DEEP: loads two stages ahead (twice the staging registers).  The overlaps stream both operands
// of K = 3 Ns^3 from memory at one or two workgroups per CU: 24^3 x 128, 112 x 112, 11.3 ms (12.1
// one stage ahead, 12.0 with single-buffered stages and 2 x 2 tiles a wave; 128 x 128 11.2 ms,
// 62 TFLOP/s).  The baryon products fill three workgroups per CU, where the registers cost
// more than the distance gains: 10.9 ms one stage ahead, 12.0 two (11.3 single-buffered).
// Small ragged sizes gain most: 46-vector baryon functions of 7^3 lines 0.113 -> 0.073 ms, 13 x 13
// overlaps on 8^3 x 16 0.27 -> 0.09 ms.
// NT: 16 x 16 tiles per wave, first .. first + NT - 1 of the workgroup tile's tm x tn (those past
// the end repeat the last one and are not stored)
template <int KT, bool PHASE, bool DEEP, int NT, class S>
__device__ __forceinline__ void tile_products(const S &s, double2 (&lds)[2][2][KT][kRow], long bt, int m0, int n0,
                                              int tm, int tn)
{
    constexpr int PER = kTM * KT / 256;
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int first = wave * NT, total = tm * tn;
    int oa[NT], ob[NT];
#pragma unroll
    for (int j = 0; j < NT; j++) {
        const int id = min(first + j, total - 1);
        oa[j] = lk * kRow + 16 * (id / tn) + lr;
        ob[j] = lk * kRow + 16 * (id % tn) + lr;
    }
    // staging: element q of a lane is e = lane + 256 q, the index along the operand's unit
    // stride fastest
    const Side sa = s.a(bt), sb = s.b(bt);
    const double2 *pa[PER], *pb[PER], *pp[PHASE ? PER : 1];
    int da[PER], db[PER];
    const bool ka = sa.sk == 1, kb = sb.sk == 1;
    auto place = [&](int q, bool kfast, int &k, int &r) {
        const int e = threadIdx.x + 256 * q;
        k = kfast ? e % KT : e / kTM;
        r = kfast ? e / KT : e % kTM;
    };
#pragma unroll
    for (int q = 0; q < PER; q++) {
        int k, r;
        place(q, ka, k, r);
        da[q] = k * kRow + r;
        pa[q] = sa.p + (long)min(m0 + r, sa.rows - 1) * sa.sr + (long)min(k, s.K - 1) * sa.sk;
        place(q, kb, k, r);
        db[q] = k * kRow + r;
        pb[q] = sb.p + (long)min(n0 + r, sb.rows - 1) * sb.sr + (long)min(k, s.K - 1) * sb.sk;
        if (PHASE) pp[q] = sb.phase + k / 3;
    }
    const int stages = (s.K + KT - 1) / KT, tail = s.K - (stages - 1) * KT;
    struct Set {
        double2 a[PER], b[PER], p[PHASE ? PER : 1];
    } v0, v1;
    auto fetch = [&](Set &v, int st) {
        const long ja = (long)st * KT * sa.sk, jb = (long)st * KT * sb.sk;
#pragma unroll
        for (int q = 0; q < PER; q++) {
            v.a[q] = pa[q][ja];
            v.b[q] = pb[q][jb];
            if (PHASE) v.p[q] = pp[q][st * (KT / 3)];
        }
    };
    // the last stage: of a K that is no multiple of KT only the rows k < tail
    auto fetch_last = [&](Set &v) {
        if (PHASE || tail == KT) {
            fetch(v, stages - 1);
            return;
        }
        const long ja = (long)(stages - 1) * KT * sa.sk, jb = (long)(stages - 1) * KT * sb.sk;
#pragma unroll
        for (int q = 0; q < PER; q++) {
            int k, r;
            place(q, ka, k, r);
            v.a[q] = make_double2(0.0, 0.0);
            if (k < tail) v.a[q] = pa[q][ja];
            place(q, kb, k, r);
            v.b[q] = make_double2(0.0, 0.0);
            if (k < tail) v.b[q] = pb[q][jb];
        }
    };
    const double cja = sa.conj ? -1.0 : 1.0;
    auto put = [&](const Set &v, int buf) {
        double2 *A = &lds[buf][0][0][0], *B = &lds[buf][1][0][0];
#pragma unroll
        for (int q = 0; q < PER; q++) {
            A[da[q]] = make_double2(v.a[q].x, cja * v.a[q].y);
            if (PHASE)
                B[db[q]] = make_double2(v.p[q].x * v.b[q].x - v.p[q].y * v.b[q].y,
                                        v.p[q].x * v.b[q].y + v.p[q].y * v.b[q].x);
            else
                B[db[q]] = v.b[q];
        }
    };
    d4 cr[NT], ci[NT];
#pragma unroll
    for (int j = 0; j < NT; j++) {
        cr[j] = d4{0.0, 0.0, 0.0, 0.0};
        ci[j] = d4{0.0, 0.0, 0.0, 0.0};
    }
    auto products = [&](int st) {
        const double2 *A = &lds[st & 1][0][0][0], *B = &lds[st & 1][1][0][0];
#pragma unroll
        for (int kk = 0; kk < KT; kk += 4) {
            double2 x[NT], y[NT];
#pragma unroll
            for (int j = 0; j < NT; j++) {
                x[j] = A[kk * kRow + oa[j]];
                y[j] = B[kk * kRow + ob[j]];
            }
#pragma unroll
            for (int j = 0; j < NT; j++) {
                cr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j].x, y[j].x, cr[j], 0, 0, 0);
                ci[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j].x, y[j].y, ci[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NT; j++) {
                cr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-x[j].y, y[j].y, cr[j], 0, 0, 0);
                ci[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j].y, y[j].x, ci[j], 0, 0, 0);
            }
        }
    };
    // (the last stage's loads stand apart in both forms: a condition on them inside the loop
    // makes the compiler wait for every load where it is issued)
    auto fetch_any = [&](Set &v, int st) {
        if (st + 1 < stages)
            fetch(v, st);
        else if (st < stages)
            fetch_last(v);
    };
    fetch_any(v0, 0);
    put(v0, 0);
    int st = 0;
    if constexpr (DEEP) {  // loads two stages ahead, in turn in v0 and v1
        fetch_any(v0, 1);
        fetch_any(v1, 2);
        __syncthreads();
        for (; st + 5 < stages; st += 2) {
            products(st);
            put(v0, (st & 1) ^ 1);
            fetch(v0, st + 3);
            __syncthreads();
            products(st + 1);
            put(v1, st & 1);
            fetch(v1, st + 4);
            __syncthreads();
        }
        for (; st < stages; st++) {
            products(st);
            if (st + 1 < stages) {
                put(v0, (st & 1) ^ 1);
                v0 = v1;
                fetch_any(v1, st + 3);
            }
            __syncthreads();
        }
    } else {
        __syncthreads();
        for (; st + 2 < stages; st++) {
            fetch(v0, st + 1);
            products(st);
            put(v0, (st & 1) ^ 1);
            __syncthreads();
        }
        if (stages > 1) {
            fetch_last(v0);
            products(stages - 2);
            put(v0, (stages - 1) & 1);
            __syncthreads();
        }
        products(stages - 1);
    }
#pragma unroll
    for (int j = 0; j < NT; j++) {
        const int id = first + j, mt = m0 + 16 * (id / tn) + lk, n = n0 + 16 * (id % tn) + lr;
        if (id >= total) break;
#pragma unroll
        for (int v = 0; v < 4; v++)
            if (mt + 4 * v < s.M && n < s.N) s.store(bt, mt + 4 * v, n, cr[j][v], ci[j][v]);
    }
}

template <int KT, bool PHASE, bool DEEP, class S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_zgemm(const S s)
{
    static_assert(KT % 4 == 0 && (!PHASE || KT % 3 == 0), "whole matrix steps and sites per stage");
    static_assert(kTM == kTN && (kTM * KT) % 256 == 0, "whole elements per lane");
    __shared__ double2 lds[2][2][KT][kRow];
    // contiguous ranges of the tiles per XCD, a batch's tiles next to each other with the
    // dimension of fewer tiles fastest (they share the other operand's rows); the tiles of
    // later batches start one further, so that the cheap corners do not pile up on the same
    // compute units (112 x 112 overlaps: 12.7 -> 11.3 ms)
    const unsigned nx = 8, per_x = gridDim.x / nx;
    const long g = blockIdx.x < per_x * nx ? (long)(blockIdx.x % nx) * per_x + blockIdx.x / nx : blockIdx.x;
    const int tiles = s.tiles_m * s.tiles_n;
    const long bt = g / tiles;
    const int tile = (int)((g - bt * tiles + bt / 8) % tiles);
    const bool mfast = s.tiles_m <= s.tiles_n;
    const int m0 = kTM * (mfast ? tile % s.tiles_m : tile / s.tiles_n);
    const int n0 = kTN * (mfast ? tile / s.tiles_m : tile % s.tiles_n);
    const int tm = min(4, (s.M - m0 + 15) >> 4), tn = min(4, (s.N - n0 + 15) >> 4);
    switch ((tm * tn + 3) >> 2) {
    case 1: tile_products<KT, PHASE, DEEP, 1>(s, lds, bt, m0, n0, tm, tn); break;
    case 2: tile_products<KT, PHASE, DEEP, 2>(s, lds, bt, m0, n0, tm, tn); break;
    case 3: tile_products<KT, PHASE, DEEP, 3>(s, lds, bt, m0, n0, tm, tn); break;
    default: tile_products<KT, PHASE, DEEP, 4>(s, lds, bt, m0, n0, tm, tn); break;
    }
}

// grid of a product (the caller checks that it fits one launch)
template <class S>
long grid_of(const S &s)
{
    return s.batches * s.tiles_m * s.tiles_n;
}

}  // namespace zg
