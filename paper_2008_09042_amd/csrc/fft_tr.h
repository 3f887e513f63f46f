// Two-radix form of the batched centred DFT along one axis (the operator F of fft.hip, whose
// data layout, fused sampling and gridding window it shares): the kernel and its launches,
// instantiated for radices up to 16 and up to 32, each with the passes of an image (fft_tr16.hip,
// fft_tr32.hip), of a gridding window (fft_tr16_grid.hip, fft_tr32_grid.hip) and of several slices
// in one launch (fft_tr16_multi.hip, fft_tr32_multi.hip) in a file of its own: a process loads a
// file's kernels with the first that it launches.
#pragma once

#include <cstring>

#include "fft_device.h"

namespace mx {

namespace {

// ---------------------------------------------------------------- two-radix transforms
// n = R0 R1 with both radices compile-time cases (2 .. 32): a thread loads the R0 inputs of a
// butterfly straight from memory into registers, transforms them, exchanges them with the
// other threads of its line through LDS once, transforms R1 of them and stores the outputs
// straight to memory.  An element crosses LDS once (a store and a load) and the workgroup
// meets one barrier, where the pass-by-pass form (fft.hip) crosses it once per radix and once
// more on the way in and out, with two barriers per radix.
//
// The chessboard signs of the centred transform are index shifts here: the plain DFT of the
// input taken from index i + n/2 (mod n), written to index k + n/2 (mod n), so they cost
// nothing (for an even radix the shift permutes a thread's own registers).
//
// Index maps: pass 0 butterfly j < R1 holds inputs i = j + r R1; its output r goes to LDS
// at (r, j); pass 1 butterfly j' < R0 reads (j', r') for r' < R1, multiplies by
// exp(-+2 pi i j' r' / n) and gives outputs k = j' + r' R0.  The LDS pitch along r is odd for
// contiguous lines (a quarter wave writes 16 consecutive j and reads 16 consecutive j', both
// conflict-free) and the tile's lines are innermost for strided ones.
//
// What bounds a pass: its bytes (16 B an element).  A 256 x 256 pass of 32 coils (33.5 MB, in
// the last-level cache) takes 9.2-10.8 us against 16-19 us pass by pass, one of 512 x 512 and
// 128 coils (537 MB) 115-133 against 148-192 us (4.0-4.7 TB/s; a copy reaches 5.0), the three
// of 120 x 100 x 90 and 8 coils (138 MB each) 19-34 against 49-67 us, a gridding pass at
// 512 x 512 and 16 coils 11-16 against 19-27 us.
// Where one line of a tile comes from and goes to.  SMP as in fft_axis_body, with the
// gridding window's passes visiting only the lines that carry work: the pad pass (4) takes
// its lines from the J wn0 window rows, the crop pass (5) from the wn1 window columns.
template <int SMP>
struct TrLine {
  const FftAxisArgs& a;
  bool valid;
  int64_t in, out;    // element offsets of index 0 of the line
  int64_t pm;         // premultiply offset (0, 4), index within a coil (1, 2)
  int64_t smp;        // sample offset of the coil (1, 2)
  int64_t st;         // stride of the line's index
  float w0;           // 1 / Phi of the line's own axis (4, 5)

  __device__ __forceinline__ TrLine(const FftAxisArgs& args, uint32_t o0, uint32_t t0, int l) : a(args) {
    st = a.inner;
    uint32_t o = o0, t = 0;
    if (a.inner == 1) {
      o = o0 + l;
      valid = o < a.tr_outer;
      if (!valid) o = o0;
    } else {
      t = t0 + l;
      valid = t < a.tr_inner;
      if (!valid) t = t0;
    }
    pm = smp = 0;
    w0 = 1.f;
    if constexpr (SMP == 4) {
      const uint32_t j = fdiv(o, a.tr_coil), r0 = o - j * (uint32_t)a.wn0;
      pm = (int64_t)r0 * a.wn1 - a.woff1;
      in = (int64_t)o * a.wn1 - a.woff1;
      out = (j * a.outer_per_coil + a.woff0 + r0) * a.n;
      w0 = a.iphi[r0];
    } else if constexpr (SMP == 5) {
      in = o * a.n * a.inner + a.woff1 + t;
      out = ((int64_t)o * a.wn0 - a.woff0) * a.wn1 + t;
      w0 = a.iphi[a.wn0 + t];
    } else {
      in = out = o * a.n * a.inner + t;
      if (SMP == 0 && a.premul) pm = (o - fdiv(o, a.tr_coil) * a.tr_coil.d) * a.n;
      if constexpr (SMP == 1 || SMP == 2 || SMP >= 8) {
        const int64_t j = fdiv(o, a.tr_coil);
        pm = in - j * a.coil_elems;
        smp = j * a.nsamples;
      }
    }
  }

  // the samples of points [q, q + C) of offsets off(r), -1 where unsampled (9, 10)
  template <int R, class Off>
  __device__ __forceinline__ void samples(int (&m)[R], Off off, int q, int C) const {
    const int32_t* inv = (SMP == 9 ? a.out_inv : a.in_inv) + pm;
#pragma unroll
    for (int r = q; r < R && r < q + C; ++r) m[r] = inv[off(r)];
  }

  // all of them ahead of the transform that forms the points, where they fit the registers
  template <int R, class Off>
  __device__ __forceinline__ void samples_ahead(int (&m)[R], Off off) const {
    if constexpr (R <= 16) {
      samples(m, off, 0, R);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // v[r] = w (E - y) for E = scale v at the sampled points, 0 elsewhere, and acc += w |E - y|^2
  // (FP64); use(r, m) sees v[r] as sample m, m < 0 where the point is unsampled (9, 10)
  template <int R, class Off, class Use>
  __device__ __forceinline__ void residual(float2 (&v)[R], int (&m)[R], float scale, double& acc, Off off, Use use) const {
    const float2* ys = a.res_y + smp;
    const float* ws = a.res_w ? a.res_w : (const float*)a.res_y;  // unweighted: loaded and not used
    const bool weighted = a.res_w;
    constexpr int C = R > 16 ? 4 : 8;  // points whose loads are in flight together: more would spill
#pragma unroll
    for (int q = 0; q < R; q += C) {
      float2 y[C];
      float w[C];
      if constexpr (R > 16) samples(m, off, q, C);
#pragma unroll
      for (int r = q; r < R && r < q + C; ++r) {
        y[r - q] = ys[max(m[r], 0)];
        w[r - q] = ws[max(m[r], 0)];
      }
#pragma unroll
      for (int r = q; r < R && r < q + C; ++r) {
        const bool on = m[r] >= 0;
        const float dx = on ? v[r].x * scale - y[r - q].x : 0.f, dy = on ? v[r].y * scale - y[r - q].y : 0.f;
        const float wr = on ? (weighted ? w[r - q] : 1.f) : 0.f;
        acc += (double)wr * ((double)dx * dx + (double)dy * dy);
        v[r] = make_float2(dx * wr, dy * wr);
        use(r, m[r]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // v[r] *= 1 where the point of offset off(r) is sampled, 0 elsewhere (8)
  template <int R, class Off>
  __device__ __forceinline__ void mask(float2 (&v)[R], Off off) const {
#pragma unroll
    for (int q = 0; q < R; q += 8) {
      int m[8];
#pragma unroll
      for (int r = q; r < R && r < q + 8; ++r) m[r - q] = a.in_inv[pm + off(r)];
#pragma unroll
      for (int r = q; r < R && r < q + 8; ++r)
        if (m[r - q] < 0) v[r] = make_float2(0.f, 0.f);
    }
  }

  // v[r] = input of the centred index idx(r), off(r) = idx(r) times the line's index stride
  template <int R, class Idx, class Off>
  __device__ __forceinline__ void load(float2 (&v)[R], Idx idx, Off off) const {
    if constexpr (SMP == 1) {
      int m[R];
#pragma unroll
      for (int r = 0; r < R; ++r) m[r] = a.in_inv[pm + off(r)];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v[r] = a.in_samples[smp + max(m[r], 0)];
      }
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (m[r] < 0) v[r] = make_float2(0.f, 0.f);
    } else if constexpr (SMP == 4) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = a.src[in + min(max(idx(r), a.woff1), a.woff1 + a.wn1 - 1)];  // clamped
#pragma unroll
      for (int q = 0; q < R; q += 8) {  // eight image values at a time: fewer registers held
        float2 x[8];
        float w[8];
#pragma unroll
        for (int r = q; r < R && r < q + 8; ++r) {
          const int i = min(max(idx(r), a.woff1), a.woff1 + a.wn1 - 1);
          x[r - q] = a.premul[pm + i];
          w[r - q] = a.iphi[a.wn0 - a.woff1 + i];
        }
#pragma unroll
        for (int r = q; r < R && r < q + 8; ++r) {
          const bool ok = idx(r) >= a.woff1 && idx(r) < a.woff1 + a.wn1;
          v[r] = ok ? cscale(cmul(v[r], x[r - q]), w0 * w[r - q]) : make_float2(0.f, 0.f);
        }
      }
    } else if constexpr (SMP == 6) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = idx(r);
        const bool ok = i >= a.woff0 && i < a.woff0 + a.wn0;
        v[r] = a.src[ok ? in + off(r) : in + (int64_t)a.woff0 * st];
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = idx(r);
        if (i < a.woff0 || i >= a.woff0 + a.wn0) v[r] = make_float2(0.f, 0.f);
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = a.src[in + off(r)];
      if (SMP == 0 && a.premul) {
        float2 x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = a.premul[pm + off(r)];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = cmul(v[r], x[r]);
      }
    }
  }

  template <int R, class Idx, class Off>
  __device__ __forceinline__ void store(const float2 (&v)[R], float scale, Idx idx, Off off) const {
    if (!valid) return;
    if constexpr (SMP == 2) {
#pragma unroll
      for (int q = 0; q < R; q += 8) {
        int m[8];
#pragma unroll
        for (int r = q; r < R && r < q + 8; ++r) m[r - q] = a.out_inv[pm + off(r)];
#pragma unroll
        for (int r = q; r < R && r < q + 8; ++r)
          if (m[r - q] >= 0) a.out_samples[smp + m[r - q]] = cscale(v[r], scale);
      }
    } else if constexpr (SMP == 5) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int k = idx(r);
        if (k >= a.woff0 && k < a.woff0 + a.wn0)
          a.crop_out[out + (int64_t)k * a.wn1] = cscale(v[r], scale * a.iphi[k - a.woff0] * w0);
      }
    } else if constexpr (SMP == 7) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int k = idx(r);
        if (k >= a.woff1 && k < a.woff1 + a.wn1) a.data[out + k] = cscale(v[r], scale);
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) a.data[out + off(r)] = cscale(v[r], scale);
    }
  }
};

// Butterfly bf of a pass with nb butterflies per line -> (line, butterfly): consecutive
// threads take consecutive butterflies of a contiguous line, consecutive lines otherwise.
__device__ __forceinline__ void tr_coords(const FftAxisArgs& a, int bf, const FastDiv& fnb, int& l, int& j) {
  if (a.inner == 1) {
    l = (int)fdiv(bf, fnb);
    j = bf - l * (int)fnb.d;
  } else {
    l = bf & (a.lines - 1);
    j = bf >> a.tr_lshift;
  }
}

struct TrLds {
  int LL, RP, JP;  // strides of line, pass-0 output digit and butterfly
};

template <int SMP, int DIR, int R>
__device__ __forceinline__ void tr_pass0(const FftAxisArgs& a, float2* lds, const TrLds& s, uint32_t o0, uint32_t t0) {
  const int nb = a.tr_r1.d, n = (int)a.n, total = nb << a.tr_lshift;
  for (int bf = threadIdx.x; bf < total; bf += blockDim.x) {
    int l, j;
    tr_coords(a, bf, a.tr_r1, l, j);
    const TrLine<SMP> line(a, o0, t0, l);
    float2 v[R];
    const int64_t b0 = j * line.st, step = nb * line.st;
    if constexpr (R % 2 == 0) {
      line.load(v, [&](int r) -> int { return j + ((r + R / 2) % R) * nb; },
                [&](int r) -> int64_t { return b0 + ((r + R / 2) % R) * step; });
    } else {
      auto idx = [&](int r) -> int {
        const int i = j + r * nb + n / 2;
        return i >= n ? i - n : i;
      };
      line.load(v, idx, [&](int r) -> int64_t { return (int64_t)idx(r) * line.st; });
    }
    tr_dft<R, DIR>(v);
    float2* d = lds + l * s.LL + j * s.JP;
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * s.RP] = v[r];
  }
}

// Offset of output r of butterfly j of pass 1 within the line's image (below 2^31 points)
template <int R>
__device__ __forceinline__ uint32_t tr_out_off(int j, int r, int nb, int n, int64_t st) {
  if constexpr (R % 2 == 0) return (uint32_t)(j + ((r + R / 2) % R) * nb) * (uint32_t)st;
  const int k = j + r * nb + n / 2;
  return (uint32_t)(k >= n ? k - n : k) * (uint32_t)st;
}

// The middle of a round trip: pass 1 of the forward transform, the mask (8) or the weighted
// residual against the measured samples (10), zero where unsampled, and pass 0 of the
// inverse, whose inputs j' + r R0 are the outputs that the thread holds.  The outputs go back
// to the LDS row that the thread read, so no barrier parts the two.
template <int SMP, int R>
__device__ __forceinline__ void tr_mask_pass(const FftAxisArgs& a, float2* lds, const float2* tw, const TrLds& s,
                                             uint32_t o0, uint32_t t0, double& acc) {
  const int nb = a.tr_r0.d, n = (int)a.n, total = nb << a.tr_lshift;
  for (int bf = threadIdx.x; bf < total; bf += blockDim.x) {
    int l, j;
    tr_coords(a, bf, a.tr_r0, l, j);
    auto off = [&](int r) { return tr_out_off<R>(j, r, nb, n, a.inner); };
    int m[R];
    if constexpr (SMP == 10) TrLine<SMP>(a, o0, t0, l).samples_ahead(m, off);
    float2* d = lds + l * s.LL + j * s.RP;
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = d[r * s.JP];
    tr_twiddle<-1, R>(v, tw, j);
    tr_dft<R, -1>(v);
    const TrLine<SMP> line(a, o0, t0, l);
    if constexpr (SMP == 8) {
      line.mask(v, off);
    } else {
      double sum = 0.0;
      line.residual(v, m, rsqrtf((float)n), sum, off, [](int, int) {});
      if (line.valid) acc += sum;
    }
    tr_dft<R, 1>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * s.JP] = v[r];
  }
}

// Pass 1 with fnb butterflies of radix R per line; the butterfly's LDS elements are rp apart
// from the next butterfly's, jp from each other.
template <int SMP, int DIR, int R>
__device__ __forceinline__ void tr_pass1(const FftAxisArgs& a, const float2* lds, const float2* tw, const FastDiv& fnb,
                                         int ll, int rp, int jp, uint32_t o0, uint32_t t0, float scale,
                                         double& acc) {
  const int nb = fnb.d, n = (int)a.n, total = nb << a.tr_lshift;
  for (int bf = threadIdx.x; bf < total; bf += blockDim.x) {
    int l, j;
    tr_coords(a, bf, fnb, l, j);
    const TrLine<SMP> line(a, o0, t0, l);
    int m[R];
    auto moff = [&](int r) { return tr_out_off<R>(j, r, nb, n, line.st); };
    if constexpr (SMP == 9) line.samples_ahead(m, moff);
    const float2* d = lds + l * ll + j * rp;
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = d[r * jp];
    tr_twiddle<DIR, R>(v, tw, j);
    tr_dft<R, DIR>(v);
    const int64_t b0 = j * line.st, step = nb * line.st;
    if constexpr (SMP == 9) {
      double sum = 0.0;
      const bool keep = line.valid && a.out_samples;
      float2* os = a.out_samples + line.smp;
      line.residual(v, m, scale, sum, moff, [&](int r, int mr) {
        if (mr >= 0 && keep) os[mr] = v[r];
      });
      if (line.valid) acc += sum;
    } else if constexpr (R % 2 == 0) {
      line.store(v, scale, [&](int r) -> int { return j + ((r + R / 2) % R) * nb; },
                 [&](int r) -> int64_t { return b0 + ((r + R / 2) % R) * step; });
    } else {
      auto idx = [&](int r) -> int {
        const int k = j + r * nb + n / 2;
        return k >= n ? k - n : k;
      };
      line.store(v, scale, idx, [&](int r) -> int64_t { return (int64_t)idx(r) * line.st; });
    }
  }
}

// BIG: radices up to 32 (about twice the registers), R0, the larger, above 16; else up to 16.
template <int SMP, int DIR, bool BIG>
__device__ __forceinline__ void fft_tr_body(const FftAxisArgs& a, uint32_t bid_in, uint32_t nbl) {
  extern __shared__ float2 lds[];
  const int n = (int)a.n, T = a.lines;
  const bool contig = a.inner == 1;
  float2* tw = lds + (contig ? T * (int)a.tr_r0.d * ((int)a.tr_r1.d | 1) : T * n);
  for (int i = threadIdx.x; i < n; i += blockDim.x) tw[i] = a.twiddle[i];
  uint32_t o0, t0 = 0;
  TrLds s;
  if (contig) {
    o0 = bid_in << a.tr_lshift;
    s.JP = 1;
    s.RP = (int)a.tr_r1.d | 1;
    s.LL = (int)a.tr_r0.d * s.RP;
  } else {
    // consecutive chunks (adjacent columns, which share cache lines) go to one XCD: the
    // hardware deals workgroups round-robin over the 8 XCDs, each with its own L2
    uint32_t bid = bid_in;
    if ((nbl & 7) == 0) bid = (bid_in & 7) * (nbl >> 3) + (bid_in >> 3);
    o0 = fdiv(bid, a.tr_chunks);
    t0 = (bid - o0 * a.tr_chunks.d) << a.tr_lshift;
    s.LL = 1;
    s.JP = T;
    s.RP = (int)a.tr_r1.d * T;
  }
#define TR_P0(R) case R: tr_pass0<SMP, DIR, R>(a, lds, s, o0, t0); break;
  if constexpr (BIG) {
    switch (a.tr_r0.d) { TR_LARGE(TR_P0) default: break; }
  } else {
    switch (a.tr_r0.d) { TR_SMALL(TR_P0) default: break; }
  }
#undef TR_P0
  __syncthreads();
  double acc = 0.0;
  if constexpr (SMP == 8 || SMP == 10) {
#define TR_M(R) case R: tr_mask_pass<SMP, R>(a, lds, tw, s, o0, t0, acc); break;
    if constexpr (BIG) {
      switch (a.tr_r1.d) { TR_SMALL(TR_M) TR_LARGE(TR_M) default: break; }
    } else {
      switch (a.tr_r1.d) { TR_SMALL(TR_M) default: break; }
    }
#undef TR_M
    __syncthreads();
    // pass 1 of the inverse: r1 butterflies of radix r0, rows and columns of the LDS tile swapped
    const float scale = SMP == 8 ? 1.f / (float)n : rsqrtf((float)n);
#define TR_P1(R) case R: tr_pass1<SMP, 1, R>(a, lds, tw, a.tr_r1, s.LL, s.JP, s.RP, o0, t0, scale, acc); break;
    if constexpr (BIG) {
      switch (a.tr_r0.d) { TR_LARGE(TR_P1) default: break; }
    } else {
      switch (a.tr_r0.d) { TR_SMALL(TR_P1) default: break; }
    }
#undef TR_P1
  } else {
    const float scale = rsqrtf((float)n);
#define TR_P1(R) case R: tr_pass1<SMP, DIR, R>(a, lds, tw, a.tr_r0, s.LL, s.RP, s.JP, o0, t0, scale, acc); break;
    if constexpr (BIG) {
      switch (a.tr_r1.d) { TR_SMALL(TR_P1) TR_LARGE(TR_P1) default: break; }
    } else {
      switch (a.tr_r1.d) { TR_SMALL(TR_P1) default: break; }
    }
#undef TR_P1
  }
  if constexpr (SMP == 9 || SMP == 10) {
    // the workgroup's loss partial, by a fixed tree
    __shared__ double red[TR_NT / 64];
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) acc += __shfl_down(acc, h);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < (int)blockDim.x / 64; ++w) acc += red[w];
      a.res_part[bid_in] = acc;
    }
  }
}

template <int SMP, int DIR, bool BIG>
__global__ __launch_bounds__(TR_NT, (BIG ? 3 : 5) - (SMP == 4 || (!BIG && SMP >= 9) ? 1 : 0)) void fft_tr_kernel(FftAxisArgs a) {
  fft_tr_body<SMP, DIR, BIG>(a, blockIdx.x, gridDim.x);
}

// Several passes (of different slices) in one launch, as fft_axis_multi_kernel (fft.hip).
template <int SMP, int DIR, bool BIG>
__global__ __launch_bounds__(TR_NT, (BIG ? 3 : 5) - (SMP == 4 || (!BIG && SMP >= 9) ? 1 : 0)) void fft_tr_multi_kernel(FftMulti m) {
  int i = 0;
  while (i + 1 < m.n && (int)blockIdx.x >= m.start[i + 1]) ++i;
  const FftAxisArgs a = m.d[i];
  fft_tr_body<SMP, DIR, BIG>(a, blockIdx.x - m.start[i], m.start[i + 1] - m.start[i]);
}

}  // namespace

// Kernel variants: what the pass reads and writes (its direction follows, except for plain
// passes), of an image and of a gridding window
#define TR_IMAGE(F) F(0, 0, -1) F(1, 0, 1) F(2, 1, 1) F(3, 2, -1) F(8, 8, -1) F(9, 9, -1) F(10, 10, -1)
#define TR_GRID(F) F(4, 4, -1) F(5, 5, 1) F(6, 6, -1) F(7, 7, 1)
// The forward pass with the residual written out (9) is built for radices up to 16 alone: with
// larger ones its launch is an error.
template <bool BIG>
constexpr bool tr_built(int smp) { return !(BIG && smp == 9); }

template <bool BIG, bool GRID>
hipError_t tr_launch_one(const FftLaunch& l, hipStream_t st) {
  const dim3 gr((unsigned)l.blocks), bl((unsigned)l.threads);
#define TR_LAUNCH(I, SMP, DIR) \
  case I:                                                                                         \
    if constexpr (tr_built<BIG>(SMP))                                                             \
      hipLaunchKernelGGL((fft_tr_kernel<SMP, DIR, BIG>), gr, bl, l.lds, st, l.a);                 \
    else                                                                                          \
      return hipErrorInvalidValue;                                                                \
    break;
  if constexpr (GRID) {
    switch (l.variant) { TR_GRID(TR_LAUNCH) default: return hipErrorInvalidValue; }
  } else {
    switch (l.variant) { TR_IMAGE(TR_LAUNCH) default: return hipErrorInvalidValue; }
  }
#undef TR_LAUNCH
  return hipGetLastError();
}

template <bool BIG>
hipError_t tr_launch_many(int variant, int threads, size_t lds, const FftMulti& m, hipStream_t st) {
  const dim3 gr((unsigned)m.start[m.n]), bl((unsigned)threads);
#define TR_LAUNCH(I, SMP, DIR) \
  case I:                                                                                         \
    if constexpr (tr_built<BIG>(SMP))                                                             \
      hipLaunchKernelGGL((fft_tr_multi_kernel<SMP, DIR, BIG>), gr, bl, lds, st, m);               \
    else                                                                                          \
      return hipErrorInvalidValue;                                                                \
    break;
  switch (variant) { TR_IMAGE(TR_LAUNCH) TR_GRID(TR_LAUNCH) default: return hipErrorInvalidValue; }
#undef TR_LAUNCH
  return hipGetLastError();
}

}  // namespace mx
