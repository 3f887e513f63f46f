// Tucker basis of the general 3D path (paper Sec. III-B, Eq. (13)): the two products next to
// the coil images, in both directions, as streams of the images.
//
// One wave holds 16 adjacent rows i1 of one i0 (all of i2, up to 128) and goes from the small
// factor T2 [J][n0][r1][r2] to the images without leaving registers: X = T2^T U1^T, whose
// result tile is as it stands the B operand of S^T = U2 X, whose tile gives each lane four
// adjacent i2 of its row.  T3 = T2 x_2 U1 is never stored.  On the way back the same tiles are
// multiplied with the coil images and summed over the coils for gx, and h = conj(x) (.) g is,
// as loaded, the A operand of h conj(U2): one read of the images gives both gradients, and the
// maps are neither written nor read.  The fragments of U2 are built once per workgroup in LDS.
//
// What bounds them: the images' traffic (one write, one read) for the BF16 split; in FP32 the
// matrix cores.  Ranks and n2 are limited by the registers that hold a wave's rows (n2 <= 128)
// and by LDS (r1, r2 <= 48); beyond, the products run as a chain of GEMMs.
//
// 120 x 100 x 90, 8 coils, ranks 20, BF16 split: maps 29.5 + 45 us as two GEMMs, 27 here;
// gradients 28 + 45 (maps again) + 33 (combination) + 40 + 34 us, here 45 + 10.  The image
// kernel runs one wave per SIMD (its tiles take most of the registers); with a branch per
// tile instead of compiled tile counts it took 56 us.
//
// Kernels and dispatch, compiled for each precision in a file of its own (tucker_rows_*.hip).
#pragma once

#include "mfma_frag.h"
#include "tucker_stream.h"

namespace mx {

struct RowsArgs {
  int64_t n1, rows16;  // rows16: row blocks of one i0
  int n0, n2, r1, r2, J, jc;
  const float2 *T2, *U1, *U2, *x, *g;
  float alpha;
  const float* alpha_dev;
  float2 *S, *gx, *Q3;
};
hipError_t tucker_maps_fp32(const RowsArgs& r, hipStream_t st);
hipError_t tucker_maps_bf16(const RowsArgs& r, hipStream_t st);
hipError_t tucker_images_fp32(const RowsArgs& r, hipStream_t st);
hipError_t tucker_images_bf16(const RowsArgs& r, hipStream_t st);
hipError_t tucker_mode1_fp32(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st);
hipError_t tucker_mode1_bf16(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st);

namespace {

constexpr int NW = 4;       // waves of a workgroup
constexpr int RANK_TILES = 3;

template <int PREC>
constexpr int fa_bytes() { return 2048; }
template <int PREC>
constexpr int fb_bytes() { return PREC == 1 ? 4096 : 2048; }

__device__ __forceinline__ float2 pick(const float2* p, int64_t i, bool ok) {
  const float2 v = p[ok ? i : 0];
  return ok ? v : make_float2(0.f, 0.f);
}

// U2 as the A operand (o = i2, k = p2), and its conjugate as the B operand (o = p2, k = i2)
template <int PREC, int PT>
__device__ __forceinline__ void build_u2(const float2* __restrict__ U2, int n2, int r2, int zt, bool fwd, bool adj,
                                         char* fa, char* fb) {
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  for (int f = wave; f < zt * PT; f += NW) {
    const int zb = f / PT, pb = f % PT;
    float2 v[4];
    if (fwd) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int z = zb * 16 + c16, p = pb * 16 + 4 * g + t;
        v[t] = pick(U2, z * r2 + p, z < n2 && p < r2);
      }
      put_frag_a<PREC>(fa, PT, zb, pb, lane, v);
    }
    if (adj) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int z = zb * 16 + 4 * g + t, p = pb * 16 + c16;
        v[t] = cconj(pick(U2, z * r2 + p, z < n2 && p < r2));
      }
      put_frag_b<PREC>(fb, PT, pb, zb, lane, v);
    }
  }
}

// Raw operands of X = T2^T U1^T at one (j, i0) and row block
template <int PT>
struct FactorRaw {
  float2 t[RANK_TILES][PT][4];  // T2[p1][p2]: A operand, o = p2, k = p1
};

template <int PT>
__device__ __forceinline__ void fetch_t2(FactorRaw<PT>& q, const float2* __restrict__ T, int r1, int r2, int p1t, int g,
                                         int c16) {
#pragma unroll
  for (int s = 0; s < RANK_TILES; ++s)
    if (s < p1t)
#pragma unroll
      for (int pb = 0; pb < PT; ++pb)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          q.t[s][pb][t] = T[min(s * 16 + 4 * g + t, r1 - 1) * r2 + min(pb * 16 + c16, r2 - 1)];
}

// X[pb] (B operand of the product with U2) from the raw operands, T2's loaded a coil ahead
template <int PREC, int PT>
__device__ __forceinline__ void make_x(typename Tile<PREC>::B (&X)[PT], const FactorRaw<PT>& q,
                                       const float2 (&u)[RANK_TILES][4], int r1, int r2, int p1t, int g, int c16) {
#pragma unroll
  for (int pb = 0; pb < PT; ++pb) {
    f32x4 cr = z4(), ci = z4();
#pragma unroll
    for (int s = 0; s < RANK_TILES; ++s)
      if (s < p1t) {
        float2 v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
          v[t] = s * 16 + 4 * g + t < r1 && pb * 16 + c16 < r2 ? q.t[s][pb][t] : make_float2(0.f, 0.f);
        Tile<PREC>::mma(cr, ci, Tile<PREC>::make_a(v), Tile<PREC>::make_b(u[s]));
      }
    X[pb] = tile_as_b<PREC>(cr, ci);
  }
}

// The same with the operands loaded when used: PT = 3 leaves no registers to hold them
template <int PREC, int PT>
__device__ __forceinline__ void load_x(typename Tile<PREC>::B (&X)[PT], const float2* __restrict__ T,
                                       const float2* __restrict__ U1, int n1, int i1, int r1, int r2, int p1t, int g,
                                       int c16) {
  f32x4 cr[PT], ci[PT];
#pragma unroll
  for (int pb = 0; pb < PT; ++pb) { cr[pb] = z4(); ci[pb] = z4(); }
#pragma unroll 1
  for (int s = 0; s < p1t; ++s) {
    float2 u[4], v[PT][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int q = s * 16 + 4 * g + t;
      u[t] = pick(U1, i1 * r1 + q, i1 < n1 && q < r1);
#pragma unroll
      for (int pb = 0; pb < PT; ++pb) v[pb][t] = pick(T, q * r2 + pb * 16 + c16, q < r1 && pb * 16 + c16 < r2);
    }
    const typename Tile<PREC>::B b = Tile<PREC>::make_b(u);
#pragma unroll
    for (int pb = 0; pb < PT; ++pb) Tile<PREC>::mma(cr[pb], ci[pb], Tile<PREC>::make_a(v[pb]), b);
  }
#pragma unroll
  for (int pb = 0; pb < PT; ++pb) X[pb] = tile_as_b<PREC>(cr[pb], ci[pb]);
}

// U1[i1][p1]: B operand, o = i1, k = p1
__device__ __forceinline__ void fetch_u1(float2 (&u)[RANK_TILES][4], const float2* __restrict__ U1, int n1, int r1,
                                         int p1t, int i1, int g) {
#pragma unroll
  for (int s = 0; s < RANK_TILES; ++s)
    if (s < p1t)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int p = s * 16 + 4 * g + t;
        u[s][t] = pick(U1, i1 * r1 + p, i1 < n1 && p < r1);
      }
}

// Keeps a value that does not change in a loop from being worked out ahead of it: the offsets
// of all tiles, held at once, would not leave the registers that the tiles need.
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A row's tiles of 16 i2, four adjacent values per lane (n2 is even; the last tile is clamped
// into the row, repeating it).
struct RowTile {
  uint32_t o, l0, l1;  // offsets of the lane's values in tile 0, and of its pairs in the last tile
  int last;
  __device__ __forceinline__ RowTile(uint32_t row, int g, int n2, int zt) {
    const int z = (zt - 1) * 16 + 4 * g;
    o = row + 4 * g;
    l0 = row + min(z, n2 - 2);
    l1 = row + min(z + 2, n2 - 2);
    last = zt - 1;
  }
  // 16-byte aligned pairs
  __device__ __forceinline__ void load(float2 (&v)[4], const float2* __restrict__ p, int zb) const {
    const float4 a = *reinterpret_cast<const float4*>(p + (zb < last ? o + zb * 16 : l0));
    const float4 b = *reinterpret_cast<const float4*>(p + (zb < last ? o + zb * 16 + 2 : l1));
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  }
  // the caller's arrays, 8-byte aligned
  __device__ __forceinline__ void load1(float2 (&v)[4], const float2* __restrict__ p, int zb) const {
    const float2 *a = p + (zb < last ? o + zb * 16 : l0), *b = p + (zb < last ? o + zb * 16 + 2 : l1);
    v[0] = a[0];
    v[1] = a[1];
    v[2] = b[0];
    v[3] = b[1];
  }
};

template <int PREC, int PT>
__global__ __launch_bounds__(64 * NW, 2) void tucker_maps_kernel(RowsArgs a) {
  extern __shared__ char lds[];
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int zt = (a.n2 + 15) / 16, p1t = (a.r1 + 15) / 16, n1 = (int)a.n1;
  build_u2<PREC, PT>(a.U2, a.n2, a.r2, zt, true, false, lds, nullptr);
  __syncthreads();
  const int64_t task = (int64_t)blockIdx.x * NW + wave;
  if (task >= a.n0 * a.rows16) return;
  const int i0 = (int)(task / a.rows16), i1 = (int)(task - i0 * a.rows16) * 16 + c16;
  const int j0 = blockIdx.y * a.jc, j1 = min(j0 + a.jc, a.J);
  float2 u[RANK_TILES][4];
  const int64_t ts = (int64_t)a.r1 * a.r2;
  FactorRaw<PT> q;
  if constexpr (PT < 3) {
    fetch_u1(u, a.U1, n1, a.r1, p1t, i1, g);
    fetch_t2<PT>(q, a.T2 + ((int64_t)j0 * a.n0 + i0) * ts, a.r1, a.r2, p1t, g, c16);
  }
  for (int j = j0; j < j1; ++j) {
    typename Tile<PREC>::B X[PT];
    if constexpr (PT < 3) {
      make_x<PREC, PT>(X, q, u, a.r1, a.r2, p1t, g, c16);
      fetch_t2<PT>(q, a.T2 + ((int64_t)min(j + 1, j1 - 1) * a.n0 + i0) * ts, a.r1, a.r2, p1t, here(g), here(c16));
    } else {
      load_x<PREC, PT>(X, a.T2 + ((int64_t)j * a.n0 + i0) * ts, a.U1, n1, i1, a.r1, a.r2, p1t, g, c16);
    }
    float2* row = a.S + (((int64_t)j * a.n0 + i0) * n1 + min(i1, n1 - 1)) * a.n2;
    for (int zb = 0; zb < zt; ++zb) {
      f32x4 cr = z4(), ci = z4();
#pragma unroll
      for (int pb = 0; pb < PT; ++pb)
        Tile<PREC>::mma(cr, ci, frag_a<PREC>(lds, PT, zb, pb, lane), X[pb]);
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = make_float2(cr[t], ci[t]);
      const int z = zb * 16 + 4 * g;  // 16-byte aligned, n2 even
      if (i1 < n1 && z < a.n2) *reinterpret_cast<float4*>(row + z) = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
      if (i1 < n1 && z + 2 < a.n2) *reinterpret_cast<float4*>(row + z + 2) = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
    }
  }
}

// ZT: tiles of i2, rounded up to even (without a branch per tile the products of one tile run
// under the next one's).  GX: with the image gradient (all coils in one wave).
template <int PREC, int PT, int ZT, bool GX>
__global__ __launch_bounds__(64 * NW, GX || ZT > 4 ? 1 : 2) void tucker_images_kernel(RowsArgs a) {
  extern __shared__ char lds[];
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int p1t = (a.r1 + 15) / 16, n1 = (int)a.n1;
  char* fb = lds + (GX ? ZT * PT * fa_bytes<PREC>() : 0);
  build_u2<PREC, PT>(a.U2, a.n2, a.r2, ZT, GX, true, lds, fb);
  __syncthreads();
  const int64_t task = (int64_t)blockIdx.x * NW + wave;
  if (task >= a.n0 * a.rows16) return;
  const int i0 = (int)(task / a.rows16), ib = (int)(task - i0 * a.rows16) * 16, i1 = ib + c16;
  const int64_t row = (int64_t)i0 * n1 + min(i1, n1 - 1);
  const int j0 = GX ? 0 : blockIdx.y * a.jc, j1 = GX ? a.J : min(j0 + a.jc, a.J);
  const int64_t ts = (int64_t)a.r1 * a.r2, js = (int64_t)a.n0 * n1 * a.n2;
  float2 u[RANK_TILES][4];
  FactorRaw<PT> q;
  if constexpr (GX && PT < 3) {
    fetch_u1(u, a.U1, n1, a.r1, p1t, i1, g);
    fetch_t2<PT>(q, a.T2 + ((int64_t)j0 * a.n0 + i0) * ts, a.r1, a.r2, p1t, g, c16);
  }
  float2 xv[2][4], sum[GX ? ZT : 1][4], cur[ZT][4];
  const float2* xs = a.x ? a.x : a.g;  // h = g: loaded and not used
  const RowTile rt((uint32_t)(row * a.n2), g, a.n2, (a.n2 + 15) / 16);
  auto fetch_x = [&](int zb) {
    RowTile rx = rt;
    rx.o = here(rx.o);
    rx.l0 = here(rx.l0);
    rx.l1 = here(rx.l1);
    rx.load1(xv[zb & 1], xs, zb);
  };
  fetch_x(0);
  fetch_x(1);
#pragma unroll
  for (int zb = 0; zb < ZT; ++zb)
    rt.load(cur[zb], a.g + j0 * js, zb);
#pragma unroll
  for (int zb = 0; zb < (GX ? ZT : 1); ++zb)
#pragma unroll
    for (int t = 0; t < 4; ++t) sum[zb][t] = make_float2(0.f, 0.f);
  for (int j = j0; j < j1; ++j) {
    const int jn = min(j + 1, j1 - 1);
    typename Tile<PREC>::B X[GX ? PT : 1];
    if constexpr (GX && PT < 3) {
      make_x<PREC, PT>(X, q, u, a.r1, a.r2, p1t, g, c16);
      fetch_t2<PT>(q, a.T2 + ((int64_t)jn * a.n0 + i0) * ts, a.r1, a.r2, p1t, here(g), here(c16));
    } else if constexpr (GX) {
      load_x<PREC, PT>(X, a.T2 + ((int64_t)j * a.n0 + i0) * ts, a.U1, n1, i1, a.r1, a.r2, p1t, g, c16);
    }
    f32x4 qr[PT], qi[PT];
#pragma unroll
    for (int pb = 0; pb < PT; ++pb) { qr[pb] = z4(); qi[pb] = z4(); }
#pragma unroll
    for (int zb = 0; zb < ZT; ++zb) {
      if constexpr (GX) {
        f32x4 cr = z4(), ci = z4();
#pragma unroll
        for (int pb = 0; pb < PT; ++pb) Tile<PREC>::mma(cr, ci, frag_a<PREC>(lds, PT, zb, pb, lane), X[pb]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          sum[zb][t] = cadd(sum[zb][t], cmulc(make_float2(cr[t], ci[t]), cur[zb][t]));
      }
      float2 h[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        h[t] = GX || a.x ? cmulc(xv[zb & 1][t], cur[zb][t]) : cur[zb][t];
        if (zb + 2 >= ZT && zb * 16 + 4 * g + t >= a.n2) h[t] = make_float2(0.f, 0.f);  // clamped loads repeat the row
      }
      const typename Tile<PREC>::A ha = Tile<PREC>::make_a(h);
#pragma unroll
      for (int pb = 0; pb < PT; ++pb) Tile<PREC>::mma(qr[pb], qi[pb], ha, frag_b<PREC>(fb, PT, pb, zb, lane));
      // the next coil's tile, as soon as this one is used up
      rt.load(cur[zb], a.g + jn * js, zb);
      if (zb + 2 < ZT) fetch_x(zb + 2);
    }
    fetch_x(0);
    fetch_x(1);
    if (a.Q3) {
      float2* out = a.Q3 + (((int64_t)j * a.n0 + i0) * n1 + ib) * a.r2;
#pragma unroll
      for (int pb = 0; pb < PT; ++pb)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (ib + 4 * g + t < n1 && pb * 16 + c16 < a.r2)
            out[(4 * g + t) * a.r2 + pb * 16 + c16] = make_float2(qr[pb][t], qi[pb][t]);
    }
  }
  if constexpr (GX) {
    const float s = a.alpha_dev ? a.alpha * *a.alpha_dev : a.alpha;
#pragma unroll
    for (int zb = 0; zb < ZT; ++zb)
      if (i1 < n1) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (zb * 16 + 4 * g + t < a.n2) a.gx[row * a.n2 + zb * 16 + 4 * g + t] = cscale(sum[zb][t], s);
      }
  }
}

// One wave per (j, i0): Q2[p1][p2] = sum_i1 conj(U1[i1][p1]) Q3[i1][p2], the fragments of U1
// (A operand, o = p1, k = i1) in LDS, Q3 loaded two steps ahead.
template <int PREC, int PT>
__global__ __launch_bounds__(64 * NW, 2) void tucker_mode1_adj_kernel(const float2* __restrict__ U1, int n1, int r1, int r2,
                                                                   int64_t tasks, const float2* __restrict__ Q3,
                                                                   float2* __restrict__ Q2) {
  extern __shared__ char lds[];
  const int lane = threadIdx.x % 64, g = lane / 16, c16 = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int steps = (n1 + 15) / 16, p1t = (r1 + 15) / 16;
  for (int f = wave; f < steps * p1t; f += NW) {
    const int s = f / p1t, pb = f % p1t;
    float2 v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = s * 16 + 4 * g + t, p = pb * 16 + c16;
      v[t] = cconj(pick(U1, (int64_t)i * r1 + p, i < n1 && p < r1));
    }
    put_frag_a<PREC>(lds, steps, pb, s, lane, v);
  }
  __syncthreads();
  const int64_t task = (int64_t)blockIdx.x * NW + wave;
  if (task >= tasks) return;
  const float2* in = Q3 + task * n1 * r2;
  struct Raw { float2 v[PT][4]; };
  auto fetch = [&](Raw& w, int s) {
#pragma unroll
    for (int pb = 0; pb < PT; ++pb)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        w.v[pb][t] = in[(int64_t)min(s * 16 + 4 * g + t, n1 - 1) * r2 + min(pb * 16 + c16, r2 - 1)];
  };
  f32x4 cr[RANK_TILES][PT], ci[RANK_TILES][PT];
#pragma unroll
  for (int q = 0; q < RANK_TILES; ++q)
#pragma unroll
    for (int pb = 0; pb < PT; ++pb) { cr[q][pb] = z4(); ci[q][pb] = z4(); }
  Raw raw[3];
  fetch(raw[0], 0);
  fetch(raw[1], min(1, steps - 1));
  for (int s0 = 0; s0 < steps; s0 += 3)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int s = s0 + k;
      fetch(raw[(k + 2) % 3], min(s + 2, steps - 1));
      __builtin_amdgcn_sched_barrier(0);
      if (s < steps) {
#pragma unroll
        for (int pb = 0; pb < PT; ++pb) {
          float2 v[4];
#pragma unroll
          for (int t = 0; t < 4; ++t)
            v[t] = s * 16 + 4 * g + t < n1 ? raw[k].v[pb][t] : make_float2(0.f, 0.f);
          const typename Tile<PREC>::B b = Tile<PREC>::make_b(v);
#pragma unroll
          for (int q = 0; q < RANK_TILES; ++q)
            if (q < p1t) Tile<PREC>::mma(cr[q][pb], ci[q][pb], frag_a<PREC>(lds, steps, q, s, lane), b);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  float2* out = Q2 + task * r1 * r2;
#pragma unroll
  for (int q = 0; q < RANK_TILES; ++q)
#pragma unroll
    for (int pb = 0; pb < PT; ++pb)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (q * 16 + 4 * g + t < r1 && pb * 16 + c16 < r2)
          out[(q * 16 + 4 * g + t) * r2 + pb * 16 + c16] = make_float2(cr[q][pb][t], ci[q][pb][t]);
}

// Coils per workgroup where they need not share one: about 1024 workgroups, four waves per
// SIMD, before a wave keeps its rows' operands for another coil.
int64_t row_grid(RowsArgs& r, bool split) {
  const int64_t gx = (r.n0 * r.rows16 + NW - 1) / NW;
  if (split) {
    int64_t y = (1024 + gx - 1) / gx;
    if (y > r.J) y = r.J;
    r.jc = (int)((r.J + y - 1) / y);
  }
  return gx;
}

template <int PREC, int PT>
hipError_t maps(RowsArgs r, hipStream_t st) {
  const int64_t gx = row_grid(r, true);
  const size_t lds = (size_t)((r.n2 + 15) / 16) * PT * fa_bytes<PREC>();
  hipLaunchKernelGGL((tucker_maps_kernel<PREC, PT>), dim3((unsigned)gx, (unsigned)((r.J + r.jc - 1) / r.jc)), dim3(64 * NW),
                     lds, st, r);
  return hipGetLastError();
}

template <int PREC, int PT, int ZT, bool GX>
hipError_t images(RowsArgs r, hipStream_t st) {
  const int64_t gx = row_grid(r, !GX);
  const size_t lds = (size_t)ZT * PT * ((GX ? fa_bytes<PREC>() : 0) + fb_bytes<PREC>());
  hipLaunchKernelGGL((tucker_images_kernel<PREC, PT, ZT, GX>), dim3((unsigned)gx, (unsigned)((r.J + r.jc - 1) / r.jc)),
                     dim3(64 * NW), lds, st, r);
  return hipGetLastError();
}

template <int PREC, int PT>
hipError_t images_any(const RowsArgs& r, hipStream_t st) {
  switch ((r.n2 + 31) / 32) {
    case 1: return r.gx ? images<PREC, PT, 2, true>(r, st) : images<PREC, PT, 2, false>(r, st);
    case 2: return r.gx ? images<PREC, PT, 4, true>(r, st) : images<PREC, PT, 4, false>(r, st);
    case 3: return r.gx ? images<PREC, PT, 6, true>(r, st) : images<PREC, PT, 6, false>(r, st);
    case 4: return r.gx ? images<PREC, PT, 8, true>(r, st) : images<PREC, PT, 8, false>(r, st);
    default: return hipErrorInvalidValue;
  }
}

template <int PREC, int PT>
hipError_t mode1_adj(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st) {
  const int64_t tasks = a.J * a.n0;
  const size_t lds = (size_t)((a.n1 + 15) / 16) * ((a.r1 + 15) / 16) * fa_bytes<PREC>();
  hipLaunchKernelGGL((tucker_mode1_adj_kernel<PREC, PT>), dim3((unsigned)((tasks + NW - 1) / NW)), dim3(64 * NW), lds, st,
                     a.U1, (int)a.n1, (int)a.r1, (int)a.r2, tasks, Q3, Q2);
  return hipGetLastError();
}

#define BY_RANK(r2, CALL)                       \
  switch (((r2) + 15) / 16) {                   \
    case 1: { constexpr int PT = 1; return CALL; } \
    case 2: { constexpr int PT = 2; return CALL; } \
    case 3: { constexpr int PT = 3; return CALL; } \
    default: return hipErrorInvalidValue;       \
  }

template <int PREC>
hipError_t maps_by_rank(const RowsArgs& r, hipStream_t st) {
  BY_RANK(r.r2, (maps<PREC, PT>(r, st)))
}
template <int PREC>
hipError_t images_by_rank(const RowsArgs& r, hipStream_t st) {
  BY_RANK(r.r2, (images_any<PREC, PT>(r, st)))
}
template <int PREC>
hipError_t mode1_by_rank(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st) {
  BY_RANK(a.r2, (mode1_adj<PREC, PT>(a, Q3, Q2, st)))
}
#undef BY_RANK

}  // namespace

}  // namespace mx
