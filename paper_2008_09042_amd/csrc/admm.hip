// Kernels of the constrained density reconstruction (paper Sec. II-C): total-variation prox,
// per-coil projection on the data-consistency balls, and the ADMM bookkeeping.
//
// TV(x) = sum_i sqrt(sum_d |x[i + e_d] - x[i]|^2) over the image (forward differences, zero at
// the last index of each axis; complex values with the real and imaginary parts coupled).
// Its prox, argmin 1/2 ||x - z||^2 + lam TV(x), runs Chambolle's dual projection steps
// (J. Math. Imaging Vis. 20, 2004) from a zero dual field P (ndim components per pixel):
//     d = div P - z / lam;   g = grad d;   P <- (P + tau g) / (1 + tau |g|),   tau = 1/(4 ndim)
// and returns x = z - lam div P, with div = -grad^H.  lam = 1 / rho is read from device memory
// (rho adapts inside the ADMM loop).  2D images run several steps per launch on tiles in LDS;
// 3D images take one launch per step, each thread recomputing d at its pixel and at its forward
// neighbours from the previous dual field (double-buffered), so that the divergence and the
// gradient need no barrier between them.
//
// Ball projection (the closed form of the paper): z_k = y_k + eps_k (w_k - y_k) /
// max(||w_k - y_k||, eps_k), with the per-coil distance accumulated in FP64 by a fixed-order
// two-stage reduction.
#include "solver.h"
#include "admm.h"

#include <utility>

namespace mx {

namespace {

constexpr int NT = 256;

inline unsigned grid_for(int64_t total, int64_t cap = 16384) {
  int64_t b = (total + NT - 1) / NT;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (unsigned)b;
}

struct Dims {
  int nd;
  int64_t n[3], stride[3], N;
};

// The pixel of a thread of a workgroup of the three-dimensional grid: the workgroup's position is
// the index, so no index is divided.
__device__ __forceinline__ bool tv_pixel(const Dims& g, int64_t& i, int (&c)[3]) {
  c[2] = blockIdx.x * blockDim.x + threadIdx.x;
  c[1] = blockIdx.y * blockDim.y + threadIdx.y;
  c[0] = blockIdx.z * blockDim.z + threadIdx.z;
  i = c[0] * g.stride[0] + c[1] * g.stride[1] + c[2];
  return c[2] < g.n[2] && c[1] < g.n[1] && c[0] < g.n[0];
}

// div P - z inv_lam at pixel i
__device__ __forceinline__ float2 tv_d_at(const Dims& g, const float2* __restrict__ P, float2 zi, float inv_lam,
                                          int64_t i, const int (&c)[3]) {
  float2 dv = make_float2(0.f, 0.f);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float2* Pd = P + d * g.N;
    if (c[d] < g.n[d] - 1) dv = cadd(dv, Pd[i]);
    if (c[d] > 0) dv = csub(dv, Pd[i - g.stride[d]]);
  }
  return make_float2(dv.x - zi.x * inv_lam, dv.y - zi.y * inv_lam);
}

__device__ __forceinline__ float2 tv_z(const float2* __restrict__ z, const float2* __restrict__ u, float uf, int64_t i) {
  float2 v = z[i];
  if (u) {
    const float2 w = u[i];
    v.x += uf * w.x;
    v.y += uf * w.y;
  }
  return v;
}

// ---- 3D images: one launch per step
__global__ __launch_bounds__(NT) void tv_step_kernel(Dims g, const float2* __restrict__ Pin, float2* __restrict__ Pout,
                                                     TvInput in, float tau) {
  const float inv_lam = in.rho ? (float)*in.rho : 1.f / in.lam;
  const float uf = in.ufac ? (float)*in.ufac : 1.f;
  int64_t i;
  int c[3];
  if (!tv_pixel(g, i, c)) return;
  const float2 di = tv_d_at(g, Pin, tv_z(in.z, in.u, uf, i), inv_lam, i, c);
  float2 gr[3];
  float m2 = 0.f;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    gr[d] = make_float2(0.f, 0.f);
    if (c[d] < g.n[d] - 1) {
      int cn[3] = {c[0], c[1], c[2]};
      cn[d] += 1;
      const int64_t k = i + g.stride[d];
      gr[d] = csub(tv_d_at(g, Pin, tv_z(in.z, in.u, uf, k), inv_lam, k, cn), di);
    }
    m2 += gr[d].x * gr[d].x + gr[d].y * gr[d].y;
  }
  const float inv = 1.f / (1.f + tau * sqrtf(m2));
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float2 pv = Pin[d * g.N + i];
    Pout[d * g.N + i] = make_float2((pv.x + tau * gr[d].x) * inv, (pv.y + tau * gr[d].y) * inv);
  }
}

// out = z - lam div P
__global__ __launch_bounds__(NT) void tv_out_kernel(Dims g, const float2* __restrict__ P, TvInput in,
                                                    float2* __restrict__ out) {
  const float lam = in.rho ? (float)(1.0 / *in.rho) : in.lam;
  int64_t i;
  int c[3];
  if (!tv_pixel(g, i, c)) return;
  const float2 zi = tv_z(in.z, in.u, in.ufac ? (float)*in.ufac : 1.f, i);
  const float2 dv = tv_d_at(g, P, make_float2(0.f, 0.f), 0.f, i, c);
  out[i] = make_float2(zi.x - lam * dv.x, zi.y - lam * dv.y);
}

// ---- 2D images: up to TV_STEPS steps per launch.  A step reads its neighbours one pixel
// around, so a workgroup that loads its TV_TILE^2 pixels with a halo of one pixel per step (one
// more above and to the left for the closing divergence) can run the steps in LDS, the valid
// region shrinking by a pixel each; only the tile itself is written.  The steps of a 256^2
// image are launch- and latency-bound: 20 steps took 20 launches of 19 us, of which most was
// 64-bit index division; one launch of five steps takes less than one of those.
constexpr int TV_TILE = 16, TV_STEPS = 5, TV_W = TV_TILE + 2 * TV_STEPS + 1;
constexpr int TV_NT = (TV_W * TV_W + 63) / 64 * 64;  // a thread per loaded pixel

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(TV_NT) void tv_tile_kernel(int n0, int n1, const float2* __restrict__ Pin,
                                                        float2* __restrict__ Pout, TvInput in, float tau, int steps,
                                                        float2* __restrict__ out) {
  __shared__ float2 P0[TV_W * TV_W], P1[TV_W * TV_W], D[TV_W * TV_W];
  const float inv_lam = in.rho ? (float)*in.rho : 1.f / in.lam;
  const float uf = in.ufac ? (float)*in.ufac : 1.f;
  const int lo = steps + 1;              // halo above and to the left
  const int W = TV_TILE + lo + steps;    // side of the loaded square
  const int64_t N = (int64_t)n0 * n1;
  const int e = threadIdx.x, ry = e / TV_W, rx = e - ry * TV_W;  // LDS rows keep the full pitch
  const int y = (int)blockIdx.y * TV_TILE - lo + ry, x = (int)blockIdx.x * TV_TILE - lo + rx;
  const bool in_sq = ry < W && rx < W, in_img = in_sq && y >= 0 && y < n0 && x >= 0 && x < n1;
  const int64_t i = in_img ? (int64_t)y * n1 + x : 0;
  const float2 z = tv_z(in.z, in.u, uf, i);
  const float2 zero = make_float2(0.f, 0.f);
  float2 p0 = zero, p1 = zero;
  if (!FIRST && in_img) {
    p0 = Pin[i];
    p1 = Pin[N + i];
  }
  if (in_sq) {
    P0[e] = p0;
    P1[e] = p1;
  }
  __syncthreads();
  // divergence at the pixel from the dual field in LDS (0 outside the image and past the square)
  auto div = [&]() {
    float2 dv = zero;
    if (y < n0 - 1) dv = cadd(dv, p0);
    if (y > 0) dv = csub(dv, ry > 0 ? P0[e - TV_W] : zero);
    if (x < n1 - 1) dv = cadd(dv, p1);
    if (x > 0) dv = csub(dv, rx > 0 ? P1[e - 1] : zero);
    return dv;
  };
  for (int s = 0; s < steps; ++s) {
    float2 d = zero;
    if (in_sq) {
      const float2 dv = div();
      d = make_float2(dv.x - z.x * inv_lam, dv.y - z.y * inv_lam);
      D[e] = d;
    }
    __syncthreads();
    if (in_sq) {
      float2 g0 = zero, g1 = zero;
      if (y < n0 - 1 && ry + 1 < W) g0 = csub(D[e + TV_W], d);
      if (x < n1 - 1 && rx + 1 < W) g1 = csub(D[e + 1], d);
      const float m2 = g0.x * g0.x + g0.y * g0.y + g1.x * g1.x + g1.y * g1.y;
      const float inv = 1.f / (1.f + tau * sqrtf(m2));
      p0 = make_float2((p0.x + tau * g0.x) * inv, (p0.y + tau * g0.y) * inv);
      p1 = make_float2((p1.x + tau * g1.x) * inv, (p1.y + tau * g1.y) * inv);
      P0[e] = p0;
      P1[e] = p1;
    }
    __syncthreads();
  }
  const int ty = ry - lo, tx = rx - lo;
  if (ty < 0 || ty >= TV_TILE || tx < 0 || tx >= TV_TILE || y >= n0 || x >= n1) return;
  if (LAST) {
    const float lam = in.rho ? (float)(1.0 / *in.rho) : in.lam;
    const float2 dv = div();
    out[i] = make_float2(z.x - lam * dv.x, z.y - lam * dv.y);
  } else {
    Pout[i] = p0;
    Pout[N + i] = p1;
  }
}

// w + uf u (u may be null): the point that a coil's ball projection starts from
__device__ __forceinline__ float2 ball_point(const float2* __restrict__ w, const float2* __restrict__ u, float uf,
                                             int64_t e) {
  return tv_z(w, u, uf, e);
}

// part[j * PB + b] = sum over block b's share of coil j of |w + uf u - y|^2 (FP64)
constexpr int PB = 64;
__global__ __launch_bounds__(NT) void coil_dist_kernel(const float2* __restrict__ w, const float2* __restrict__ u,
                                                       const double* __restrict__ ufac, const float2* __restrict__ y,
                                                       int64_t M, double* __restrict__ part) {
  __shared__ double s[NT];
  const int j = blockIdx.y;
  const int64_t j0 = (int64_t)j * M;
  const float uf = ufac ? (float)*ufac : 1.f;
  double acc = 0.0;
  for (int64_t m = blockIdx.x * (int64_t)NT + threadIdx.x; m < M; m += (int64_t)PB * NT) {
    const float2 wv = ball_point(w, u, uf, j0 + m), yv = y[j0 + m];
    const double dx = (double)wv.x - (double)yv.x, dy = (double)wv.y - (double)yv.y;
    acc += dx * dx + dy * dy;
  }
  s[threadIdx.x] = acc;
  for (int h = NT / 2; h > 0; h >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
  }
  if (threadIdx.x == 0) part[(int64_t)j * PB + blockIdx.x] = s[0];
}

// z = y + eps (w + uf u - y) / max(dist, eps) for coil blockIdx.y, whose distance every
// workgroup sums from its PB partials; t (optional) = z - uf u - w, the data part of the
// p-update's right side
__global__ __launch_bounds__(NT) void ball_kernel(const float2* __restrict__ w, const float2* __restrict__ u,
                                                  const double* __restrict__ ufac, const float2* __restrict__ y,
                                                  const float* __restrict__ eps, const double* __restrict__ part,
                                                  int64_t M, float2* __restrict__ z, float2* __restrict__ t) {
  __shared__ double s[PB];
  const int j = blockIdx.y;
  if (threadIdx.x < PB) s[threadIdx.x] = part[(int64_t)j * PB + threadIdx.x];
  for (int h = PB / 2; h > 0; h >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
  }
  __syncthreads();
  const double dist = sqrt(s[0]), ej = (double)eps[j], den = dist > ej ? dist : ej;
  const float f = den > 0.0 ? (float)(ej / den) : 0.f;
  const float uf = ufac ? (float)*ufac : 1.f;
  const int64_t j0 = (int64_t)j * M;
  for (int64_t m = blockIdx.x * (int64_t)NT + threadIdx.x; m < M; m += (int64_t)gridDim.x * NT) {
    const int64_t e = j0 + m;
    const float2 yv = y[e], wv = ball_point(w, u, uf, e);
    const float2 zv = make_float2(yv.x + f * (wv.x - yv.x), yv.y + f * (wv.y - yv.y));
    z[e] = zv;
    if (t) {
      const float2 uv = u[e], fv = w[e];
      t[e] = make_float2((zv.x - uf * uv.x) - fv.x, (zv.y - uf * uv.y) - fv.y);
    }
  }
}

// 256 FP64 values in LDS -> s[0], by a fixed tree
__device__ __forceinline__ void tree256(double* s) {
  for (int h = NT / 2; h > 0; h >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
  }
  __syncthreads();
}

// The p-update's start: b = g + z0 - uf u0 - p; x = 0, r = d = b, partials of <r, r>
__global__ __launch_bounds__(NT) void admm_start_kernel(const float2* __restrict__ g, const float2* __restrict__ z0,
                                                        const float2* __restrict__ u0, const double* __restrict__ ufac,
                                                        const float2* __restrict__ p, int64_t n, float2* __restrict__ x,
                                                        float2* __restrict__ r, float2* __restrict__ d,
                                                        double* __restrict__ part) {
  __shared__ double s[NT];
  const float uf = (float)*ufac;
  double acc = 0.0;
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 gv = g[e], zv = z0[e], uv = u0[e], pv = p[e];
    const float2 v = make_float2(((gv.x + zv.x) - uf * uv.x) - pv.x, ((gv.y + zv.y) - uf * uv.y) - pv.y);
    x[e] = make_float2(0.f, 0.f);
    r[e] = v;
    d[e] = v;
    acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
  }
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// u = uf u + A p - z over the image block (p, z0, u0; n0 entries) and the data block (Fp, zk,
// uk; n1 entries); t = zk - zkp over the data block; partials of ||A p - z||^2
__global__ __launch_bounds__(NT) void admm_dual_kernel(const float2* __restrict__ p, const float2* __restrict__ z0,
                                                       float2* __restrict__ u0, int64_t n0,
                                                       const float2* __restrict__ Fp, const float2* __restrict__ zk,
                                                       const float2* __restrict__ zkp, float2* __restrict__ uk,
                                                       float2* __restrict__ t, int64_t n1,
                                                       const double* __restrict__ ufac, double* __restrict__ part) {
  __shared__ double s[NT];
  const float uf = (float)*ufac;
  double acc = 0.0;
  for (int64_t q = blockIdx.x * (int64_t)NT + threadIdx.x; q < n0 + n1; q += (int64_t)gridDim.x * NT) {
    const bool img = q < n0;
    const int64_t e = img ? q : q - n0;
    const float2 av = img ? p[e] : Fp[e], zv = img ? z0[e] : zk[e];
    float2* u = img ? u0 : uk;
    const float2 uv = u[e];
    u[e] = make_float2((uf * uv.x + av.x) - zv.x, (uf * uv.y + av.y) - zv.y);
    const float2 dv = csub(av, zv);
    acc += (double)dv.x * (double)dv.x + (double)dv.y * (double)dv.y;
    if (!img) t[e] = csub(zv, zkp[e]);
  }
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// partials of ||g + z0 - z0p||^2, the dual residual's square before rho
__global__ __launch_bounds__(NT) void admm_dres_kernel(const float2* __restrict__ g, const float2* __restrict__ z0,
                                                       const float2* __restrict__ z0p, int64_t n,
                                                       double* __restrict__ part) {
  __shared__ double s[NT];
  double acc = 0.0;
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    const float2 gv = g[e], zv = z0[e], zp = z0p[e];
    const float2 v = make_float2((gv.x + zv.x) - zp.x, (gv.y + zv.y) - zp.y);
    acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
  }
  s[threadIdx.x] = acc;
  tree256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// hist = (rho, r, s) with r and s / rho the roots of the partials' sums; residual balancing of
// rho.  *ufac is the factor that the duals' next readers apply.
__global__ __launch_bounds__(NT) void admm_rho_kernel(const double* __restrict__ part_r, const double* __restrict__ part_s,
                                                      double* __restrict__ rho, double* __restrict__ ufac,
                                                      double* __restrict__ hist) {
  __shared__ double s[NT];
  static_assert(DOT_BLOCKS == NT, "one partial per thread");
  s[threadIdx.x] = part_r[threadIdx.x];
  tree256(s);
  const double r2 = s[0];
  __syncthreads();
  s[threadIdx.x] = part_s[threadIdx.x];
  tree256(s);
  if (threadIdx.x != 0) return;
  const double r = sqrt(r2), ds = *rho * sqrt(s[0]);
  if (hist) {
    hist[0] = *rho;
    hist[1] = r;
    hist[2] = ds;
  }
  if (r > 10.0 * ds) {
    *rho *= 2.0;
    *ufac = 0.5;
  } else if (ds > 10.0 * r) {
    *rho *= 0.5;
    *ufac = 2.0;
  } else {
    *ufac = 1.0;
  }
}

// z0 = u0 = 0 (n0 entries), zk = uk = 0 (n1 entries); rho, ufac = 1
__global__ void admm_init_kernel(float2* __restrict__ z0, float2* __restrict__ u0, int64_t n0, float2* __restrict__ zk,
                                 float2* __restrict__ uk, int64_t n1, double rho0, double* __restrict__ rho,
                                 double* __restrict__ ufac) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *rho = rho0;
    *ufac = 1.0;
  }
  const float2 zero = make_float2(0.f, 0.f);
  for (int64_t e = blockIdx.x * (int64_t)NT + threadIdx.x; e < n0 + n1; e += (int64_t)gridDim.x * NT) {
    (e < n0 ? z0 : zk - n0)[e] = zero;
    (e < n0 ? u0 : uk - n0)[e] = zero;
  }
}

// Axes are aligned at the last: a 2D image has n[0] = 1.
Dims make_dims(int nd, const int64_t* n) {
  Dims g;
  g.nd = nd;
  g.N = 1;
  for (int d = 0; d < 3; ++d) g.n[d] = d >= 3 - nd ? n[d - (3 - nd)] : 1;
  for (int d = 2; d >= 0; --d) {
    g.stride[d] = g.N;
    g.N *= g.n[d];
  }
  return g;
}

}  // namespace

hipError_t tv_prox_launch(int nd, const int64_t* n, const TvInput& in, int iters, float2* P, float2* P2, float2* x,
                          hipStream_t st) {
  const Dims g = make_dims(nd, n);
  const float tau = 1.f / (4.f * (float)nd);
  if (!in.rho && !(in.lam > 0.f)) return copy_split_launch(x, nullptr, in.z, nullptr, g.N, 0, st);  // prox of 0
  float2 *pin = P, *pout = P2;
  if (nd == 2) {
    const dim3 gr((unsigned)((g.n[2] + TV_TILE - 1) / TV_TILE), (unsigned)((g.n[1] + TV_TILE - 1) / TV_TILE));
    const int n0 = (int)g.n[1], n1 = (int)g.n[2];
    int k = 0;
    do {
      const int s = iters - k < TV_STEPS ? iters - k : TV_STEPS;
      const bool first = k == 0, last = k + s >= iters;
      if (first && last)
        hipLaunchKernelGGL((tv_tile_kernel<true, true>), gr, dim3(TV_NT), 0, st, n0, n1, pin, pout, in, tau, s, x);
      else if (first)
        hipLaunchKernelGGL((tv_tile_kernel<true, false>), gr, dim3(TV_NT), 0, st, n0, n1, pin, pout, in, tau, s, x);
      else if (last)
        hipLaunchKernelGGL((tv_tile_kernel<false, true>), gr, dim3(TV_NT), 0, st, n0, n1, pin, pout, in, tau, s, x);
      else
        hipLaunchKernelGGL((tv_tile_kernel<false, false>), gr, dim3(TV_NT), 0, st, n0, n1, pin, pout, in, tau, s, x);
      std::swap(pin, pout);
      k += s;
    } while (k < iters);
    return hipGetLastError();
  }
  // A wave along the last axis, the rest of the workgroup's threads along the others: at most 64
  // pixels of the last axis, and no more of the last two than they hold, rounded up to a power of
  // two.  Always (64, 4, 1) left a short axis' threads without pixels: 500 x 480 x 2, 20 steps 4814 -> 272 us,
  // 400 x 400 x 4 3558 -> 422.
  auto side = [](int64_t n, int most) {
    int b = 1;
    while (b < n && b < most) b *= 2;
    return b;
  };
  // A small image is bound by latency: a workgroup with a short last axis is halved, down to a wave, while
  // there are few of them (20 steps at 32 x 30 x 16 134 -> 111 us, 18 x 36 x 10 144 -> 126, 64 x 30 x 24
  // 138 -> 123; (64, 4, 1) takes 119, 130 and 126).
  const int bx = side(g.n[2], 64);
  int by, bz;
  dim3 gr;
  for (int threads = NT;; threads /= 2) {
    by = side(g.n[1], threads / bx);
    bz = threads / (bx * by);
    gr = dim3((unsigned)((g.n[2] + bx - 1) / bx), (unsigned)((g.n[1] + by - 1) / by), (unsigned)((g.n[0] + bz - 1) / bz));
    if (bx == 64 || threads == 64 || (int64_t)gr.x * gr.y * gr.z >= 384) break;
  }
  const dim3 bl(bx, by, bz);
  hipError_t e = zero_split_launch(P, nullptr, (int64_t)nd * g.N, 0, st);
  if (e != hipSuccess) return e;
  for (int k = 0; k < iters; ++k) {
    hipLaunchKernelGGL(tv_step_kernel, gr, bl, 0, st, g, pin, pout, in, tau);
    std::swap(pin, pout);
  }
  hipLaunchKernelGGL(tv_out_kernel, gr, bl, 0, st, g, pin, in, x);
  return hipGetLastError();
}

hipError_t ball_project_launch(const float2* w, const float2* u, const double* ufac, const float2* y, const float* eps,
                               int64_t M, int J, double* part, float2* z, float2* t, hipStream_t st) {
  if (M * J == 0) return hipSuccess;
  hipLaunchKernelGGL(coil_dist_kernel, dim3(PB, J), dim3(NT), 0, st, w, u, ufac, y, M, part);
  hipLaunchKernelGGL(ball_kernel, dim3(grid_for(M, 64), J), dim3(NT), 0, st, w, u, ufac, y, eps, part, M, z, t);
  return hipGetLastError();
}

int ball_part_doubles(int J) { return J * PB + J; }

hipError_t admm_init_launch(float2* z0, float2* u0, int64_t n0, float2* zk, float2* uk, int64_t n1, double rho0,
                            double* rho, double* ufac, hipStream_t st) {
  hipLaunchKernelGGL(admm_init_kernel, dim3(grid_for(n0 + n1)), dim3(NT), 0, st, z0, u0, n0, zk, uk, n1, rho0, rho,
                     ufac);
  return hipGetLastError();
}

hipError_t admm_start_launch(const float2* g, const float2* z0, const float2* u0, const double* ufac, const float2* p,
                             int64_t n, float2* x, float2* r, float2* d, double* part, hipStream_t st) {
  hipLaunchKernelGGL(admm_start_kernel, dim3(DOT_BLOCKS), dim3(NT), 0, st, g, z0, u0, ufac, p, n, x, r, d, part);
  return hipGetLastError();
}

hipError_t admm_dual_launch(const float2* p, const float2* z0, float2* u0, int64_t n0, const float2* Fp,
                            const float2* zk, const float2* zkp, float2* uk, float2* t, int64_t n1, const double* ufac,
                            double* part, hipStream_t st) {
  hipLaunchKernelGGL(admm_dual_kernel, dim3(DOT_BLOCKS), dim3(NT), 0, st, p, z0, u0, n0, Fp, zk, zkp, uk, t, n1, ufac,
                     part);
  return hipGetLastError();
}

hipError_t admm_dres_launch(const float2* g, const float2* z0, const float2* z0p, int64_t n, double* part,
                            hipStream_t st) {
  hipLaunchKernelGGL(admm_dres_kernel, dim3(DOT_BLOCKS), dim3(NT), 0, st, g, z0, z0p, n, part);
  return hipGetLastError();
}

hipError_t admm_rho_launch(const double* part_r, const double* part_s, double* rho, double* ufac, double* hist,
                           hipStream_t st) {
  hipLaunchKernelGGL(admm_rho_kernel, dim3(1), dim3(NT), 0, st, part_r, part_s, rho, ufac, hist);
  return hipGetLastError();
}

}  // namespace mx
