// Vector kernels of the Gauss-Newton step (paper Sec. II-B, Eq. (6)): the normal operator
// J^H W J + diag(lambda) is applied with the operator kernels; conjugate gradients around it
// need complex axpy, a row weighting, and inner products.
//
// A CG vector v = (v_x, v_c) is an image block of N complex values and a coefficient block
// of J K values.  The work vectors live contiguously in the workspace ([N | J K]); the
// caller's solution blocks are two pointers.  Every kernel takes the two blocks as one
// virtual vector of N + J K entries.
//
// Inner products Re <a, b> = Re sum conj(a) b are accumulated in FP64: every thread sums its
// grid-stride entries in order, the workgroup reduces its 256 sums by a fixed tree, and the
// DOT_BLOCKS partials are reduced by the same tree wherever the sum is read.  No atomics: the
// result does not depend on timing.  The CG scalars stay in device memory in FP64, so a CG
// solve runs with no host synchronisation and can be captured into a graph.
//
// The vectors of a CG step are short (0.5 MB at 256^2, 4 MB at 96 x 80 x 64) and each kernel
// over them costs its launch and ramp (2-5 us), so a step takes three of them: the shift of
// the operator's result with the partials of <d, q>; x, r and the partials of <r, r>; d.
// Every workgroup of the last two forms the step's scalars itself from the 256 partials.
#include "solver.h"

namespace mx {

namespace {

constexpr int NT = 256;

inline unsigned grid_for(int64_t total, int64_t cap = 16384) {
  int64_t b = (total + NT - 1) / NT;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (unsigned)b;
}

struct Split {
  float2* p0;  // entries [0, n0)
  float2* p1;  // entries [n0, n0 + n1)
  int64_t n0, n1;
  __device__ float2& at(int64_t e) const { return e < n0 ? p0[e] : p1[e - n0]; }
};

struct CSplit {
  const float2* p0;
  const float2* p1;
  int64_t n0, n1;
  __device__ float2 at(int64_t e) const { return e < n0 ? p0[e] : p1[e - n0]; }
};

__global__ void caxpy_kernel(float2* __restrict__ y, const float2* __restrict__ x, float a, int64_t n) {
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 v = x[e];
    float2 o = y[e];
    o.x += a * v.x;
    o.y += a * v.y;
    y[e] = o;
  }
}

__global__ void weight_rows_kernel(float2* __restrict__ u, const float* __restrict__ w, int64_t M, int J) {
  const int64_t total = M * J;
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    const float s = w[e % M];
    float2 v = u[e];
    u[e] = make_float2(v.x * s, v.y * s);
  }
}

__global__ void copy_split_kernel(Split dst, CSplit src) {
  const int64_t n = dst.n0 + dst.n1;
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT)
    dst.at(e) = src.at(e);
}

__global__ void zero_split_kernel(Split dst) {
  const int64_t n = dst.n0 + dst.n1;
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT)
    dst.at(e) = make_float2(0.f, 0.f);
}

// 256 FP64 values in LDS -> s[0], by a fixed tree
__device__ __forceinline__ void tree256(double* s) {
  for (int h = NT / 2; h > 0; h >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
  }
  __syncthreads();
}

// Sum of DOT_BLOCKS partials, the same value in every thread (s: NT doubles of LDS).
__device__ __forceinline__ double sum_parts(const double* __restrict__ part, double* s) {
  static_assert(DOT_BLOCKS == NT, "one partial per thread");
  __syncthreads();
  s[threadIdx.x] = part[threadIdx.x];
  tree256(s);
  return s[0];
}

// (q0 | q1) += (l0 d0 | l1 d1); with part, the partials of <d, q> for the new q
template <bool DOT>
__global__ __launch_bounds__(NT) void axpy_dot_kernel(Split q, CSplit d, float l0, float l1, double* __restrict__ part) {
  __shared__ double s[NT];
  const int64_t n = q.n0 + q.n1;
  double acc = 0.0;
#pragma unroll 4
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float l = e < q.n0 ? l0 : l1;
    const float2 dv = d.at(e);
    float2 qv = q.at(e);
    qv.x += l * dv.x;
    qv.y += l * dv.y;
    q.at(e) = qv;
    if (DOT) acc += (double)dv.x * (double)qv.x + (double)dv.y * (double)qv.y;
  }
  if (!DOT) return;
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// x = 0, r = d = b and the partials of <r, r>
__global__ __launch_bounds__(NT) void cg_start_kernel(Split x, CSplit b, float2* __restrict__ r, float2* __restrict__ d,
                                                      double* __restrict__ part) {
  __shared__ double s[NT];
  const int64_t n = x.n0 + x.n1;
  double acc = 0.0;
#pragma unroll 4
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 v = b.at(e);
    x.at(e) = make_float2(0.f, 0.f);
    r[e] = v;
    d[e] = v;
    acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
  }
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// alpha = rho / <d, q> (0 when <d, q> = 0); x += alpha d, r -= alpha q, partials of <r, r>
__global__ __launch_bounds__(NT) void cg_xr_kernel(Split x, float2* __restrict__ r, const float2* __restrict__ d,
                                                   const float2* __restrict__ q, const double* __restrict__ rho,
                                                   const double* __restrict__ part_dq, double* __restrict__ part_rr) {
  __shared__ double s[NT];
  const double dq = sum_parts(part_dq, s);
  const float a = (float)(dq != 0.0 ? *rho / dq : 0.0);
  const int64_t n = x.n0 + x.n1;
  double acc = 0.0;
#pragma unroll 4
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 dv = d[e], qv = q[e];
    float2& xv = x.at(e);
    xv.x += a * dv.x;
    xv.y += a * dv.y;
    float2 rv = r[e];
    rv.x -= a * qv.x;
    rv.y -= a * qv.y;
    r[e] = rv;
    acc += (double)rv.x * (double)rv.x + (double)rv.y * (double)rv.y;
  }
  __syncthreads();  // s[0] read by all
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = s[0];
}

// rho_new = <r, r> from its partials, beta = rho_new / rho (0 when rho = 0): d = r + beta d; the
// first workgroup keeps rho_new in *rho_next (not rho, which the others may still read) and rr
__global__ __launch_bounds__(NT) void cg_d_kernel(float2* __restrict__ d, const float2* __restrict__ r, int64_t n,
                                                  const double* __restrict__ rho, const double* __restrict__ part_rr,
                                                  double* __restrict__ rho_next, double* __restrict__ rr) {
  __shared__ double s[NT];
  const double rho_new = sum_parts(part_rr, s);
  const float b = (float)(*rho != 0.0 ? rho_new / *rho : 0.0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *rho_next = rho_new;
    if (rr) *rr = rho_new;
  }
#pragma unroll 4
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 rv = r[e];
    const float2 dv = d[e];
    d[e] = make_float2(rv.x + b * dv.x, rv.y + b * dv.y);
  }
}

// *out = sum of the partials, and *out2 if given
__global__ __launch_bounds__(NT) void sum_parts_kernel(const double* __restrict__ part, double* __restrict__ out,
                                                       double* __restrict__ out2) {
  __shared__ double s[NT];
  const double v = sum_parts(part, s);
  if (threadIdx.x == 0) {
    *out = v;
    if (out2) *out2 = v;
  }
}

// out[e] = sum_i part[i * stride + e] in index order (plain FP32 adds)
__global__ void sum_rows_kernel(float2* __restrict__ out, const float2* __restrict__ part, int n, int64_t stride,
                                int64_t len) {
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < len; e += (int64_t)gridDim.x * NT) {
    float2 s = part[e];
    for (int i = 1; i < n; ++i) {
      const float2 v = part[(int64_t)i * stride + e];
      s.x = s.x + v.x;
      s.y = s.y + v.y;
    }
    out[e] = s;
  }
}

__global__ void sum_doubles_kernel(double* __restrict__ out, const double* __restrict__ part, int n, int64_t stride) {
  if (threadIdx.x != 0) return;
  double s = part[0];
  for (int i = 1; i < n; ++i) s += part[(int64_t)i * stride];
  *out = s;
}

}  // namespace

hipError_t caxpy_launch(float2* y, const float2* x, float a, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(caxpy_kernel, dim3(grid_for(n)), dim3(NT), 0, st, y, x, a, n);
  return hipGetLastError();
}

hipError_t weight_rows_launch(float2* u, const float* w, int64_t M, int J, hipStream_t st) {
  if (M * J <= 0) return hipSuccess;
  hipLaunchKernelGGL(weight_rows_kernel, dim3(grid_for(M * J)), dim3(NT), 0, st, u, w, M, J);
  return hipGetLastError();
}

hipError_t copy_split_launch(float2* d0, float2* d1, const float2* s0, const float2* s1, int64_t n0, int64_t n1,
                             hipStream_t st) {
  if (n0 + n1 <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_split_kernel, dim3(grid_for(n0 + n1)), dim3(NT), 0, st, Split{d0, d1, n0, n1},
                     CSplit{s0, s1, n0, n1});
  return hipGetLastError();
}

hipError_t zero_split_launch(float2* d0, float2* d1, int64_t n0, int64_t n1, hipStream_t st) {
  if (n0 + n1 <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_split_kernel, dim3(grid_for(n0 + n1)), dim3(NT), 0, st, Split{d0, d1, n0, n1});
  return hipGetLastError();
}

hipError_t axpy_dot_launch(float2* q0, float2* q1, const float2* d0, const float2* d1, float l0, float l1, int64_t n0,
                           int64_t n1, double* part, hipStream_t st) {
  const Split q{q0, q1, n0, n1};
  const CSplit d{d0, d1, n0, n1};
  if (part)
    hipLaunchKernelGGL(axpy_dot_kernel<true>, dim3(DOT_BLOCKS), dim3(NT), 0, st, q, d, l0, l1, part);
  else if (n0 + n1 > 0)
    hipLaunchKernelGGL(axpy_dot_kernel<false>, dim3(grid_for(n0 + n1)), dim3(NT), 0, st, q, d, l0, l1, part);
  return hipGetLastError();
}

hipError_t cg_start_launch(float2* x0, float2* x1, const float2* b0, const float2* b1, int64_t n0, int64_t n1, float2* r,
                           float2* d, double* part, hipStream_t st) {
  hipLaunchKernelGGL(cg_start_kernel, dim3(DOT_BLOCKS), dim3(NT), 0, st, Split{x0, x1, n0, n1}, CSplit{b0, b1, n0, n1},
                     r, d, part);
  return hipGetLastError();
}

hipError_t cg_xr_launch(float2* x0, float2* x1, int64_t n0, int64_t n1, float2* r, const float2* d, const float2* q,
                        const double* rho, const double* part_dq, double* part_rr, hipStream_t st) {
  hipLaunchKernelGGL(cg_xr_kernel, dim3(DOT_BLOCKS), dim3(NT), 0, st, Split{x0, x1, n0, n1}, r, d, q, rho, part_dq,
                     part_rr);
  return hipGetLastError();
}

hipError_t cg_d_launch(float2* d, const float2* r, int64_t n, const double* rho, const double* part_rr,
                       double* rho_next, double* rr, hipStream_t st) {
  hipLaunchKernelGGL(cg_d_kernel, dim3(grid_for(n, 1024)), dim3(NT), 0, st, d, r, n, rho, part_rr, rho_next, rr);
  return hipGetLastError();
}

hipError_t sum_parts_launch(const double* part, double* out, double* out2, hipStream_t st) {
  hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(NT), 0, st, part, out, out2);
  return hipGetLastError();
}

hipError_t sum_rows_launch(float2* out, const float2* part, int n, int64_t stride, int64_t len, hipStream_t st) {
  if (len <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sum_rows_kernel, dim3(grid_for(len)), dim3(NT), 0, st, out, part, n, stride, len);
  return hipGetLastError();
}

hipError_t sum_doubles_launch(double* out, const double* part, int n, int64_t stride, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sum_doubles_kernel, dim3(1), dim3(64), 0, st, out, part, n, stride);
  return hipGetLastError();
}

}  // namespace mx
