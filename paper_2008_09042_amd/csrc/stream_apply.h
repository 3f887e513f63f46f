// Dense basis apply, S_j = B c_j (paper Sec. II-B, Eq. (5)), and the image gradient
// gx = s sum_j conj(B c_j) (.) g_j (Sec. II-B, J_G^H), as streams of the basis B [N][K].
//
// Both read B once (2 J real products per element of B: far below the matrix cores' ridge
// point at few coils), so they are built for the stream.  S^T tiles of 16 coils x 16 rows of B:
// the A operand is c, whose fragments a workgroup builds once in LDS (2 KiB per 16 coils and
// K16 step), the B operand 16 rows of B, lane l (row l % 16, group g = l / 16) holding
// B[n][k0 + 4g .. +3], loaded straight into registers three steps ahead of their use.  Eight
// waves per workgroup, each with RB row blocks and all (up to 64) coils; the loads are
// unconditional (addresses clamped into the lane's own row), since a guarded load makes every
// use wait for all loads in flight.  An accumulator tile holds S[4g + r][n0 + l % 16], so a
// store is 128 contiguous bytes of each of four coils.
//
// The image gradient consumes its tiles in registers: S is neither written nor read back, and
// the maps' 2 J N complex words leave the backward pass.
//
// 256 x 256, 32 coils, 200 columns (105 MB of basis), BF16-split: apply 34 + 3 (c fragments in
// their own launch) -> 25.5 us; rebuilt maps and coil combination 34 + 3 + 11 -> 25.8 us.
//
// Kernels and dispatch; the maps and the image gradient of each precision are compiled in a file
// of their own (stream_maps_*.hip, stream_gx_*.hip), so that a process loads the code that it runs.
#pragma once

#include "mfma_frag.h"
#include "dense_stream.h"

namespace mx {

// One call of either product; S for the maps, g, alpha, alpha_dev and gx for the image gradient.
struct ApplyCall {
  const float2* B;
  int64_t N;
  int K;
  const float2* c;
  int J;
  float2* S;
  const float2* g;
  float alpha;
  const float* alpha_dev;
  float2* gx;
  int nw;  // waves per workgroup
};
hipError_t stream_maps_fp32(const ApplyCall& a, hipStream_t st);
hipError_t stream_maps_bf16(const ApplyCall& a, hipStream_t st);
hipError_t stream_gx_fp32(const ApplyCall& a, hipStream_t st);
hipError_t stream_gx_bf16(const ApplyCall& a, hipStream_t st);

namespace {

constexpr int NT = 512;                 // most threads of a workgroup
constexpr int CF_BYTES = 2048;          // one fragment of c in LDS
constexpr int CF_MAX = 128 * 1024;      // LDS of the c fragments held at a time

template <int PREC>
__device__ __forceinline__ typename Tile<PREC>::A cf_load(const uint4* cf, int f, int lane) {
  const uint4* p = cf + (size_t)f * 128 + lane;
  if constexpr (PREC == 1) {
    return typename Tile<1>::A{__builtin_bit_cast(u16x8, p[0]), __builtin_bit_cast(u16x8, p[64])};
  } else {
    const float4 u = __builtin_bit_cast(float4, p[0]), w = __builtin_bit_cast(float4, p[64]);
    return typename Tile<0>::A{{make_float2(u.x, u.y), make_float2(u.z, u.w), make_float2(w.x, w.y),
                                make_float2(w.z, w.w)}};
  }
}

template <int PREC>
__device__ __forceinline__ void cf_store(uint4* cf, int f, int lane, const float2 (&v)[4]) {
  uint4* p = cf + (size_t)f * 128 + lane;
  const typename Tile<PREC>::A a = Tile<PREC>::make_a(v);
  if constexpr (PREC == 1) {
    p[0] = __builtin_bit_cast(uint4, a.h);
    p[64] = __builtin_bit_cast(uint4, a.l);
  } else {
    p[0] = __builtin_bit_cast(uint4, make_float4(v[0].x, v[0].y, v[1].x, v[1].y));
    p[64] = __builtin_bit_cast(uint4, make_float4(v[2].x, v[2].y, v[3].x, v[3].y));
  }
}

// VEC 2: rows of B are 16-byte aligned (K even), else 1.  GX: the image gradient.  FEW: K <= 64,
// whose rows stay in the four load stages for every coil group (fetched again per group, they
// were seven times the work: 150 us instead of 78 at 512 x 512, 128 coils, 16 columns).
template <int PREC, int JB, int RB, int VEC, bool GX, bool FEW>
__global__ __launch_bounds__(NT) void stream_apply_kernel(const float2* __restrict__ B, int64_t N, int K,
                                                          const float2* __restrict__ c, int J, int cs, int all,
                                                          float2* __restrict__ S, const float2* __restrict__ gin,
                                                          float alpha, const float* __restrict__ alpha_dev,
                                                          float2* __restrict__ gx) {
  extern __shared__ uint4 cf[];
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), nw = blockDim.x / 64;
  const int64_t n0 = ((int64_t)blockIdx.x * nw + wave) * (16 * RB);
  const int steps = (K + 15) / 16;
  const float2* rowp[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int64_t n = n0 + rb * 16 + c16;
    rowp[rb] = B + (n < N ? n : N - 1) * K;
  }
  struct Raw { float2 v[4]; };
  auto fetch = [&](Raw (&raw)[RB], int s) {
    const int k = s * 16 + 4 * g;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if constexpr (VEC == 2) {
        const float4 a = *reinterpret_cast<const float4*>(rowp[rb] + min(k, K - 2));
        const float4 b = *reinterpret_cast<const float4*>(rowp[rb] + min(k + 2, K - 2));
        raw[rb].v[0] = make_float2(a.x, a.y);
        raw[rb].v[1] = make_float2(a.z, a.w);
        raw[rb].v[2] = make_float2(b.x, b.y);
        raw[rb].v[3] = make_float2(b.z, b.w);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) raw[rb].v[t] = rowp[rb][min(k + t, K - 1)];
      }
    }
  };
  float2 gsum[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) gsum[rb] = make_float2(0.f, 0.f);
  const int jgs = (J + 16 * JB - 1) / (16 * JB);
  // fragments f of coil group jg, steps s0 + f / JB
  auto build = [&](int jg, int s0, int ns, uint4* dst) {
    for (int f = wave; f < ns * JB; f += nw) {
      const int s = s0 + f / JB, j = jg * 16 * JB + (f % JB) * 16 + c16, k = s * 16 + 4 * g;
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool ok = j < J && k + t < K;
        const float2 w = c[ok ? (int64_t)j * K + k + t : 0];
        v[t] = ok ? w : make_float2(0.f, 0.f);
      }
      cf_store<PREC>(dst, f, lane, v);
    }
  };
  // GX: the coil images of the tiles, loaded a coil group ahead
  struct Gv { float2 v[GX ? RB : 1][GX ? JB : 1][4]; };
  auto fetch_g = [&](Gv& q, int jg) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t n = n0 + rb * 16 + c16;
          const int j = min((jg * JB + jb) * 16 + 4 * g + r, J - 1);
          q.v[GX ? rb : 0][GX ? jb : 0][r] = gin[(int64_t)j * N + (n < N ? n : N - 1)];
        }
  };
  Raw raw[4][RB];
  if constexpr (FEW) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < steps) fetch(raw[u], u);
  }
  Gv gv, gnext;
  if constexpr (GX) fetch_g(gv, 0);
  for (int jg = GX ? 0 : blockIdx.y; jg < (GX ? jgs : (int)blockIdx.y + 1); ++jg) {
    const int j0 = jg * 16 * JB;
    f32x4 cr[RB][JB], ci[RB][JB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) { cr[rb][jb] = z4(); ci[rb][jb] = z4(); }
    for (int s0 = 0; s0 < steps; s0 += cs) {
      const int ns = min(cs, steps - s0);
      if constexpr (!FEW) {
#pragma unroll
        for (int u = 0; u < 3; ++u) fetch(raw[u], s0 + min(u, ns - 1));
      }
      if (GX && s0 == 0) fetch_g(gnext, min(jg + 1, jgs - 1));
      const uint4* cfj = cf;
      if (GX && all) {  // every coil group's fragments at once
        if (jg == 0) {
          for (int q = 0; q < jgs; ++q) build(q, 0, steps, cf + (size_t)q * steps * JB * 128);
          __syncthreads();
        }
        cfj = cf + (size_t)jg * steps * JB * 128;
      } else {
        if (s0 > 0 || jg > 0) __syncthreads();  // the fragments held are used up
        build(jg, s0, ns, cf);
        __syncthreads();
      }
      auto compute = [&](const Raw (&rw)[RB], int s) {
        typename Tile<PREC>::A a[JB];
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) a[jb] = cf_load<PREC>(cfj, s * JB + jb, lane);
        const int k = (s0 + s) * 16 + 4 * g;
        const bool tail = (s0 + s) * 16 + 16 > K;  // columns past K: the clamped loads repeat the row
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          float2 v[4] = {rw[rb].v[0], rw[rb].v[1], rw[rb].v[2], rw[rb].v[3]};
          if (tail) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (k + t >= K) v[t] = make_float2(0.f, 0.f);
          }
          const typename Tile<PREC>::B b = Tile<PREC>::make_b(v);
#pragma unroll
          for (int jb = 0; jb < JB; ++jb) Tile<PREC>::mma(cr[rb][jb], ci[rb][jb], a[jb], b);
        }
      };
      if constexpr (FEW) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u < ns) compute(raw[u], u);
        continue;
      }
      for (int s = 0; s < ns; s += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          fetch(raw[(u + 3) & 3], s0 + min(s + u + 3, ns - 1));
          __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
          if (s + u < ns) compute(raw[u], s + u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int64_t n = n0 + rb * 16 + c16;
#pragma unroll
      for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = j0 + jb * 16 + 4 * g + r;
          const float2 v = make_float2(cr[rb][jb][r], ci[rb][jb][r]);
          if constexpr (GX) {
            if (j < J) gsum[rb] = cadd(gsum[rb], cmulc(v, gv.v[rb][jb][r]));
          } else {
            if (j < J && n < N) S[(int64_t)j * N + n] = v;
          }
        }
    }
    if constexpr (GX) gv = gnext;
  }
  if constexpr (GX) {
    const float s = alpha_dev ? alpha * *alpha_dev : alpha;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float2 v = gsum[rb];
      v.x += __shfl_xor(v.x, 16);
      v.y += __shfl_xor(v.y, 16);
      v.x += __shfl_xor(v.x, 32);
      v.y += __shfl_xor(v.y, 32);
      const int64_t n = n0 + rb * 16 + c16;
      if (g == 0 && n < N) gx[n] = cscale(v, s);
    }
  }
}

// The maps of at most 16 columns (one K16 step) and 32 coils over many rows: a workgroup that takes its rows and
// ends is mostly its start, the fragments of c behind a barrier.  Here a wave goes through row
// blocks with the rows of four in flight, and c's operands stay in registers.  BF16-split, the kernel
// above against this one: 1500 x 1500, 2 coils, 4 columns 43.4 -> 32.8 us; 2000 x 2000, 1 coil, 4
// columns 70.1 -> 49.9 (c's fragments in their own launch: 38.8 and 57.9); 1024 x 1024, 20 coils, 8
// columns 55.8 -> 36.8.
constexpr int NARROW_GRID = 512;  // two workgroups per compute unit; 1024: 33.4, 50.2 and 43.0 us
template <int PREC, int JB, int VEC>
__global__ __launch_bounds__(NT) void stream_narrow_kernel(const float2* __restrict__ B, int64_t N, int K,
                                                           const float2* __restrict__ c, int J, float2* __restrict__ S) {
  constexpr int RB = 2;
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16, k = 4 * g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), nw = blockDim.x / 64;
  const int64_t stride = (int64_t)gridDim.x * nw * (16 * RB);
  int64_t n0 = ((int64_t)blockIdx.x * nw + wave) * (16 * RB);
  struct Raw { float2 v[RB][4]; };
  auto fetch = [&](Raw& raw, int64_t first) {  // clamped into B: past the last row, that row again
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int64_t n = first + rb * 16 + c16;
      const float2* row = B + (n < N ? n : N - 1) * K;
      if constexpr (VEC == 2) {
        const float4 a = *reinterpret_cast<const float4*>(row + min(k, K - 2));
        const float4 b = *reinterpret_cast<const float4*>(row + min(k + 2, K - 2));
        raw.v[rb][0] = make_float2(a.x, a.y);
        raw.v[rb][1] = make_float2(a.z, a.w);
        raw.v[rb][2] = make_float2(b.x, b.y);
        raw.v[rb][3] = make_float2(b.z, b.w);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) raw.v[rb][t] = row[min(k + t, K - 1)];
      }
    }
  };
  Raw raw[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) fetch(raw[u], n0 + u * stride);
  typename Tile<PREC>::A a[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb) {
    const int j = jb * 16 + c16;
    float2 v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bool ok = j < J && k + t < K;
      const float2 w = c[ok ? (int64_t)j * K + k + t : 0];
      v[t] = ok ? w : make_float2(0.f, 0.f);
    }
    a[jb] = Tile<PREC>::make_a(v);
  }
  for (;;) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (n0 >= N) return;
      f32x4 cr[RB][JB], ci[RB][JB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float2 v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = k + t < K ? raw[u].v[rb][t] : make_float2(0.f, 0.f);
        const typename Tile<PREC>::B b = Tile<PREC>::make_b(v);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
          cr[rb][jb] = ci[rb][jb] = z4();
          Tile<PREC>::mma(cr[rb][jb], ci[rb][jb], a[jb], b);
        }
      }
      fetch(raw[u], n0 + 4 * stride);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int64_t n = n0 + rb * 16 + c16;
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = jb * 16 + 4 * g + r;
            if (j < J && n < N) S[(int64_t)j * N + n] = make_float2(cr[rb][jb][r], ci[rb][jb][r]);
          }
      }
      n0 += stride;
    }
  }
}

template <int PREC, int JB, int RB, int VEC, bool GX, bool FEW>
hipError_t launch_few(const ApplyCall& a, hipStream_t st) {
  const int steps = (a.K + 15) / 16;
  int cs = CF_MAX / (JB * CF_BYTES);
  if (cs > steps) cs = steps;
  const int jgs = (a.J + 16 * JB - 1) / (16 * JB);
  const int all = GX && (size_t)jgs * steps * JB * CF_BYTES <= (size_t)CF_MAX ? 1 : 0;
  const int64_t rows = (int64_t)a.nw * 16 * RB;
  const dim3 gr((unsigned)((a.N + rows - 1) / rows), GX ? 1u : (unsigned)jgs);
  hipLaunchKernelGGL((stream_apply_kernel<PREC, JB, RB, VEC, GX, FEW>), gr, dim3(64 * a.nw), (size_t)(all ? jgs * steps : cs) * JB * CF_BYTES, st,
                     a.B, a.N, a.K, a.c, a.J, cs, all, a.S, a.g, a.alpha, a.alpha_dev, a.gx);
  return hipGetLastError();
}

template <int PREC, int JB, int VEC>
hipError_t launch_narrow(const ApplyCall& a, hipStream_t st) {
  hipLaunchKernelGGL((stream_narrow_kernel<PREC, JB, VEC>), dim3(NARROW_GRID), dim3(NT), 0, st, a.B, a.N, a.K, a.c, a.J, a.S);
  return hipGetLastError();
}

template <int PREC, int JB, int RB, int VEC, bool GX>
hipError_t launch(const ApplyCall& a, hipStream_t st) {
  return a.K <= 64 ? launch_few<PREC, JB, RB, VEC, GX, true>(a, st) : launch_few<PREC, JB, RB, VEC, GX, false>(a, st);
}

// Rows per workgroup: 256 (eight waves of two row blocks), 128 (of one) or 64 (four waves of
// one), whichever leaves the busiest compute unit the fewest rows; the larger at equal rows,
// for its loads per wave and fewer builds of the c fragments.  The image gradient takes coils
// in groups of 32 at most, so that the next group's coil images fit the registers.
template <int PREC, bool GX>
hipError_t dispatch(ApplyCall a, hipStream_t st) {
  bool wide = false;
  int64_t best = INT64_MAX;
  for (int rows = 256; rows >= 64; rows /= 2) {
    const int64_t load = ((a.N + rows - 1) / rows + 255) / 256 * rows;
    if (load < best) {
      best = load;
      wide = rows == 256;
      a.nw = rows == 64 ? 4 : 8;
    }
  }
  const bool vec = a.K % 2 == 0 && (reinterpret_cast<uintptr_t>(a.B) & 15u) == 0;
  const int jb = a.J <= 16 ? 0 : a.J <= 32 || GX ? 1 : 2;
  // Few columns, and four blocks of 32 rows for every wave of the narrow kernel: 1000 x 1000, 1 coil, 4
  // columns 19.9 -> 16.6 us, 512 x 512, 2 coils, 4 columns 6.6 -> 7.6.  Past 32 coils it has no
  // registers for the rows in flight (1024 x 1024, 40 coils, 16 columns 107 -> 116).
  if constexpr (!GX) {
    if (jb < 2 && a.K <= 16 && a.N >= (int64_t)4 * NARROW_GRID * NT / 64 * 32) {
      if (jb == 0) return vec ? launch_narrow<PREC, 1, 2>(a, st) : launch_narrow<PREC, 1, 1>(a, st);
      return vec ? launch_narrow<PREC, 2, 2>(a, st) : launch_narrow<PREC, 2, 1>(a, st);
    }
  }
  switch (jb * 4 + (wide ? 2 : 0) + (vec ? 1 : 0)) {
    case 0: return launch<PREC, 1, 1, 1, GX>(a, st);
    case 1: return launch<PREC, 1, 1, 2, GX>(a, st);
    case 2: return launch<PREC, 1, 2, 1, GX>(a, st);
    case 3: return launch<PREC, 1, 2, 2, GX>(a, st);
    case 4: return launch<PREC, 2, 1, 1, GX>(a, st);
    case 5: return launch<PREC, 2, 1, 2, GX>(a, st);
    case 6: return launch<PREC, 2, 2, 1, GX>(a, st);
    case 7: return launch<PREC, 2, 2, 2, GX>(a, st);
    default: break;
  }
  if constexpr (!GX) {
    switch ((wide ? 2 : 0) + (vec ? 1 : 0)) {
      case 0: return launch<PREC, 4, 1, 1, GX>(a, st);
      case 1: return launch<PREC, 4, 1, 2, GX>(a, st);
      case 2: return launch<PREC, 4, 2, 1, GX>(a, st);
      default: return launch<PREC, 4, 2, 2, GX>(a, st);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace mx
