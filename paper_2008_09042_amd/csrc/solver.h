// Launchers of the Gauss-Newton / conjugate-gradient vector kernels (solver.hip).
#pragma once

#include "common.h"

namespace mx {

constexpr int DOT_BLOCKS = 256;  // FP64 partial sums per inner product

// y += a x over n complex entries
hipError_t caxpy_launch(float2* y, const float2* x, float a, int64_t n, hipStream_t st);
// u[j][m] *= w[m]
hipError_t weight_rows_launch(float2* u, const float* w, int64_t M, int J, hipStream_t st);
// (d0 | d1) = (s0 | s1), blocks of n0 and n1 entries
hipError_t copy_split_launch(float2* d0, float2* d1, const float2* s0, const float2* s1, int64_t n0, int64_t n1,
                             hipStream_t st);
hipError_t zero_split_launch(float2* d0, float2* d1, int64_t n0, int64_t n1, hipStream_t st);
// (q0 | q1) += (l0 d0 | l1 d1); with part (DOT_BLOCKS doubles) the partials of Re <d, q>
hipError_t axpy_dot_launch(float2* q0, float2* q1, const float2* d0, const float2* d1, float l0, float l1, int64_t n0,
                           int64_t n1, double* part, hipStream_t st);
// (x0 | x1) = 0, r = d = (b0 | b1), partials of <r, r>
hipError_t cg_start_launch(float2* x0, float2* x1, const float2* b0, const float2* b1, int64_t n0, int64_t n1, float2* r,
                           float2* d, double* part, hipStream_t st);
// (x0 | x1) += alpha d, r -= alpha q with alpha = *rho / <d, q> (0 if that is 0); partials of <r, r>
hipError_t cg_xr_launch(float2* x0, float2* x1, int64_t n0, int64_t n1, float2* r, const float2* d, const float2* q,
                        const double* rho, const double* part_dq, double* part_rr, hipStream_t st);
// d = r + beta d with beta = <r, r> / *rho (0 if *rho is 0); *rho_next = <r, r>, and *rr if given
hipError_t cg_d_launch(float2* d, const float2* r, int64_t n, const double* rho, const double* part_rr,
                       double* rho_next, double* rr, hipStream_t st);
// *out = sum of DOT_BLOCKS partials, and *out2 if given
hipError_t sum_parts_launch(const double* part, double* out, double* out2, hipStream_t st);
// out = sum over i < n of part[i * stride .. + len) in index order; the same for FP64 scalars
hipError_t sum_rows_launch(float2* out, const float2* part, int n, int64_t stride, int64_t len, hipStream_t st);
hipError_t sum_doubles_launch(double* out, const double* part, int n, int64_t stride, hipStream_t st);

}  // namespace mx
