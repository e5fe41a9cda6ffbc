// Batched Laplacian / Chebyshev launchers shared by the eigensolver.
#pragma once

#include "laph_impl.h"

// workgroups of one slice in a launch with sums
int lap_blocks(const Geom &g);
// out = alpha Lap(in) + beta in + gamma prev on every slice; vectors of slice t start at
// ptr + t * stride (complex elements).  sums (may be null) takes, per slice and workgroup, Re
// and Im of <dot, out> and |out|^2: sums[(t * lap_blocks + block) * 3 + k], dot with its stride
void lap_fused(laph_ctx *c, const double2 *us, const double2 *in, long in_stride, const double2 *prev,
               long prev_stride, double2 *out, long out_stride, double alpha, double beta, double gamma,
               const double2 *dot = nullptr, long dot_stride = 0, double *sums = nullptr);

// out = T_order(B) in with B = 1 + 2/(lamL - lamC) (Lap + lamC); w0, w1 scratch; sums (may be
// null) as above with dot = in
void cheb_apply(laph_ctx *c, const double2 *us, const double2 *in, long in_stride, double2 *out, long out_stride,
                double2 *w0, double2 *w1, long w_stride, double lamL, double lamC, int order, double *sums);
