// Dense basis adjoint, gc_j = s B^H h_j (the basis block of J_G^H, paper Sec. II-B), as a
// stream of the basis B [N][K], with h_j = conj(x) (.) g_j formed on the way.
//
// gc^T[k][j] = sum_n conj(B[n][k]) h[j][n] reduces over the long dimension.  The A operand
// (tile rows k, reduction n) is conj(B) read down four rows per lane, two adjacent columns at
// a time where rows are 16-byte aligned (256 contiguous bytes of a row per 16 lanes; the two
// columns belong to two tiles); the B operand is h, 32 contiguous bytes per lane.  A
// workgroup's eight waves are one, two or four groups of 16 AKB columns times groups of rows; a wave
// loads the next 16 rows while it multiplies the current ones.  Every load is unconditional
// (addresses clamped): a guarded load makes every use wait for all loads in flight.  The row
// groups' tiles are added through LDS in a fixed order, one partial per workgroup, and a
// second kernel sums the partials (no atomics).
//
// 256 x 256, 32 coils, 200 columns (105 MB of basis), BF16-split: 59 + 5 us (tiled GEMM and its
// split sum) -> 31 + 4 us.
//
// Kernels and dispatch, compiled for each precision in a file of its own (stream_adjoint_*.hip).
#pragma once

#include "mfma_frag.h"
#include "adjoint_geom.h"
#include "dense_stream.h"

namespace mx {

// c [J][K] = s B^H h, or of conj(x) (.) h when x is given; part holds the row chunks' partials.
struct AdjCall {
  const float2* B;
  int64_t N;
  int K;
  const float2 *h, *x;
  int J;
  float2* part;
  int max_chunks;
  float alpha;
  const float* alpha_dev;
  float2* c;
};
hipError_t stream_adjoint_fp32(const AdjCall& a, hipStream_t st);
hipError_t stream_adjoint_bf16(const AdjCall& a, hipStream_t st);

namespace {

constexpr int NW = ADJ_WAVES, NT = 64 * NW;

template <int PREC, int JB, int AKB, int VEC, bool X>
__global__ __launch_bounds__(NT) void stream_adjoint_kernel(const float2* __restrict__ B, int64_t N, int K,
                                                            const float2* __restrict__ h, const float2* __restrict__ x,
                                                            int J, int64_t chunk, int kwl, int jgs,
                                                            float2* __restrict__ part) {
  extern __shared__ f32x4 red[];  // [row group][tile][re, im][lane]
  // the wave's index in a scalar register: its rows and branches are uniform
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int kw = 1 << kwl, RW = NW >> kwl, kgi = wave & (kw - 1), rg = wave >> kwl;
  const int jg = blockIdx.y % jgs, ks = blockIdx.y / jgs;
  const int64_t ch = blockIdx.x;
  const int k0 = (ks * kw + kgi) * 16 * AKB, j0 = jg * 16 * JB;
  const int64_t r0 = ch * chunk + rg * 16;
  const int steps = (int)(chunk / (16 * RW));
  // column of tile kb and tile row i: 16 kb + i, or, two columns per load, 32 (kb / 2) + 2 i + kb % 2
  constexpr int NL = AKB / VEC;  // loads per row
  int col[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) col[q] = min(k0 + 16 * VEC * q + VEC * c16, K - VEC);
  int64_t hrow[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb) hrow[jb] = (int64_t)min(j0 + 16 * jb + c16, J - 1) * N;
  struct Raw {
    float2 b[AKB][4], h[JB][4], x[X ? 4 : 1];
  };
  auto fetch4 = [&](const float2* p, int last, float2 (&v)[4]) {  // p[4g .. 4g + 3], up to p[last]
    if constexpr (VEC == 2) {
      const float4 a = *reinterpret_cast<const float4*>(p + min(4 * g, last - 1));
      const float4 b = *reinterpret_cast<const float4*>(p + min(4 * g + 2, last - 1));
      v[0] = make_float2(a.x, a.y);
      v[1] = make_float2(a.z, a.w);
      v[2] = make_float2(b.x, b.y);
      v[3] = make_float2(b.z, b.w);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = p[min(4 * g + t, last)];
    }
  };
  // rows as 32-bit offsets from the step's first (a scalar): B's fit, 16 rows of K < 2^24 columns
  auto fetch = [&](Raw& r, int i) {
    const int64_t n = min(r0 + (int64_t)i * 16 * RW, N - 1);  // uniform
    const int last = (int)min((int64_t)15, N - 1 - n);
    const float2* rowb = B + n * K;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t row = (uint32_t)min(4 * g + t, last) * (uint32_t)K;
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        if constexpr (VEC == 2) {
          const float4 a = *reinterpret_cast<const float4*>(rowb + row + col[q]);
          r.b[2 * q][t] = make_float2(a.x, a.y);
          r.b[2 * q + 1][t] = make_float2(a.z, a.w);
        } else {
          r.b[q][t] = rowb[row + col[q]];
        }
      }
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) fetch4(h + hrow[jb] + n, last, r.h[jb]);
    if constexpr (X) fetch4(x + n, last, r.x);
    __builtin_amdgcn_sched_barrier(0);  // the step's loads stay together, ahead of the products
  };
  f32x4 cr[AKB][JB], ci[AKB][JB];
#pragma unroll
  for (int kb = 0; kb < AKB; ++kb)
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) { cr[kb][jb] = z4(); ci[kb][jb] = z4(); }
  auto compute = [&](const Raw& r, int i) {
    const int64_t n = r0 + (int64_t)i * 16 * RW;
    const bool tail = n + 16 > N;  // rows past N count as zero
    typename Tile<PREC>::B hb[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v[t] = X ? cmulc(r.x[X ? t : 0], r.h[jb][t]) : r.h[jb][t];
      }
      if (tail) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (n + 4 * g + t >= N) v[t] = make_float2(0.f, 0.f);
      }
      hb[jb] = Tile<PREC>::make_b(v);
    }
#pragma unroll
    for (int kb = 0; kb < AKB; ++kb) {
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = cconj(r.b[kb][t]);
      const typename Tile<PREC>::A a = Tile<PREC>::make_a(v);
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) Tile<PREC>::mma(cr[kb][jb], ci[kb][jb], a, hb[jb]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  Raw ra, rb;
  fetch(ra, 0);
  for (int i = 0; i < steps; i += 2) {
    fetch(rb, min(i + 1, steps - 1));
    compute(ra, i);
    fetch(ra, min(i + 2, steps - 1));
    if (i + 1 < steps) compute(rb, i + 1);
  }
  // the row groups' tiles, halved until group 0 holds the sum
  constexpr int TS = AKB * JB * 2 * 64;
  for (int half = RW / 2; half > 0; half /= 2) {
    if (rg >= half && rg < 2 * half) {
      f32x4* d = red + (size_t)((rg - half) * kw + kgi) * TS + lane;
#pragma unroll
      for (int kb = 0; kb < AKB; ++kb)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
          d[(kb * JB + jb) * 128] = cr[kb][jb];
          d[(kb * JB + jb) * 128 + 64] = ci[kb][jb];
        }
    }
    __syncthreads();
    if (rg < half) {
      const f32x4* d = red + (size_t)(rg * kw + kgi) * TS + lane;
#pragma unroll
      for (int kb = 0; kb < AKB; ++kb)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
          cr[kb][jb] += d[(kb * JB + jb) * 128];
          ci[kb][jb] += d[(kb * JB + jb) * 128 + 64];
        }
    }
    __syncthreads();
  }
  if (rg != 0) return;
#pragma unroll
  for (int jb = 0; jb < JB; ++jb) {
    const int j = j0 + 16 * jb + c16;
    if (j >= J) continue;
    float2* dst = part + (ch * J + j) * K;
#pragma unroll
    for (int kb = 0; kb < AKB; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * g + r;
        const int k = VEC == 2 ? k0 + 32 * (kb / 2) + 2 * i + kb % 2 : k0 + 16 * kb + i;
        if (k < K) dst[k] = make_float2(cr[kb][jb][r], ci[kb][jb][r]);
      }
  }
}

// out[j][k] = s * sum over chunks of part[chunk][j][k], s = alpha (* alpha_dev).  RG threads
// per output each sum every RG-th chunk in four interleaved chains, and the RG sums are added
// through LDS in a fixed order: the result does not depend on timing.
constexpr int RNT = 256, RG = 16;
__global__ __launch_bounds__(RNT) void stream_reduce_kernel(const float2* __restrict__ part, int nchunk, int64_t JK,
                                                            float alpha, const float* __restrict__ alpha_dev,
                                                            float2* __restrict__ out) {
  constexpr int OPB = RNT / RG;
  __shared__ float2 red[RG][OPB];
  const int lo = threadIdx.x % OPB, grp = threadIdx.x / OPB;
  const int64_t e = (int64_t)blockIdx.x * OPB + lo;
  float2 a0 = make_float2(0.f, 0.f), a1 = a0, a2 = a0, a3 = a0;
  if (e < JK) {
    int c = grp;
    for (; c + 3 * RG < nchunk; c += 4 * RG) {
      a0 = cadd(a0, part[(int64_t)c * JK + e]);
      a1 = cadd(a1, part[(int64_t)(c + RG) * JK + e]);
      a2 = cadd(a2, part[(int64_t)(c + 2 * RG) * JK + e]);
      a3 = cadd(a3, part[(int64_t)(c + 3 * RG) * JK + e]);
    }
    for (; c < nchunk; c += RG) a0 = cadd(a0, part[(int64_t)c * JK + e]);
  }
  red[grp][lo] = cadd(cadd(a0, a1), cadd(a2, a3));
  __syncthreads();
  if (grp != 0 || e >= JK) return;
  float2 v = red[0][lo];
  for (int q = 1; q < RG; ++q) v = cadd(v, red[q][lo]);
  float sc = alpha;
  if (alpha_dev) sc *= *alpha_dev;
  out[e] = cscale(v, sc);
}

template <int PREC, int JB, int AKB, int VEC, bool X>
hipError_t launch(const AdjCall& a, const AdjGeom& q, hipStream_t st) {
  const int RW = NW >> q.kwl;
  const size_t lds = (size_t)(RW / 2) * (1 << q.kwl) * AKB * JB * 2 * 64 * sizeof(f32x4);
  hipLaunchKernelGGL((stream_adjoint_kernel<PREC, JB, AKB, VEC, X>), dim3((unsigned)q.nchunk, (unsigned)(q.jgs * q.ks)),
                     dim3(NT), lds, st, a.B, a.N, a.K, a.h, a.x, a.J, q.chunk, q.kwl, q.jgs, a.part);
  return hipGetLastError();
}

template <int PREC, int VEC, bool X>
hipError_t dispatch(const AdjCall& a, const AdjGeom& q, hipStream_t st) {
  switch (q.JB * 8 + q.AKB) {
    case 10: return launch<PREC, 1, 2, VEC, X>(a, q, st);
    case 12: return launch<PREC, 1, 4, VEC, X>(a, q, st);
    case 18: return launch<PREC, 2, 2, VEC, X>(a, q, st);
    case 20: return launch<PREC, 2, 4, VEC, X>(a, q, st);
    default: return launch<PREC, 4, 2, VEC, X>(a, q, st);
  }
}

template <int PREC>
hipError_t adjoint(const AdjCall& a, hipStream_t st) {
  const AdjGeom q = adj_geom(a.N, a.K, a.J, a.max_chunks);
  auto odd = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
  const bool vec = a.K % 2 == 0 && a.N % 2 == 0 && !odd(a.B) && !odd(a.h) && !odd(a.x);
  hipError_t e;
  switch ((vec ? 2 : 0) + (a.x ? 1 : 0)) {
    case 0: e = dispatch<PREC, 1, false>(a, q, st); break;
    case 1: e = dispatch<PREC, 1, true>(a, q, st); break;
    case 2: e = dispatch<PREC, 2, false>(a, q, st); break;
    default: e = dispatch<PREC, 2, true>(a, q, st); break;
  }
  if (e != hipSuccess) return e;
  const int64_t JK = (int64_t)a.J * a.K;
  const unsigned rb = (unsigned)((JK + RNT / RG - 1) / (RNT / RG));
  hipLaunchKernelGGL(stream_reduce_kernel, dim3(rb), dim3(RNT), 0, st, a.part, q.nchunk, JK, a.alpha, a.alpha_dev, a.c);
  return hipGetLastError();
}

}  // namespace

}  // namespace mx
