// The last pass of F_s^H with the coil sum of J_G^H (paper Sec. II-B) in it:
//
//   out[row][k] = sum_j conj(S_j[row][k]) (F^H g_j[row])[k]
//
// along the last (contiguous) axis, two radices of at most 16 (fft_tr.h).  A workgroup takes a
// row of every coil, a tile of coils at a time: each thread holds the same outputs of one line
// of the tile throughout, so the sum over tiles stays in registers and one over the tile's
// lines, through LDS in a fixed order, ends it.  The images after the pass are neither written
// nor read: two of the five passes over the coil stack that the transform and a separate
// combination make.  The next tile's points and the maps are loaded ahead of the products that
// use them.  256^2, 32 coils: 12.9 + 6.6 us -> 13.1.
#include "fft_tr.h"

namespace mx {

namespace {

template <int R>
__device__ __forceinline__ int centred(int j, int r, int nb, int n) {
  if constexpr (R % 2 == 0) return j + ((r + R / 2) % R) * nb;
  const int k = j + r * nb + n / 2;
  return k >= n ? k - n : k;
}

template <int R>
__device__ __forceinline__ void combine_load(float2 (&v)[16], const float2* __restrict__ p, int j, int nb, int n) {
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = p[centred<R>(j, r, nb, n)];
}

template <int R>
__device__ __forceinline__ void combine_pass0(const float2 (&in)[16], float2* d, int rp) {
  float2 v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = in[r];
  tr_dft<R, 1>(v);
#pragma unroll
  for (int r = 0; r < R; ++r) d[r * rp] = v[r];
}

template <int R>
__device__ __forceinline__ void combine_pass1(float2 (&sum)[16], const float2 (&s)[16], const float2* d,
                                              const float2* tw, int j, float scale, bool ok) {
  float2 v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = d[r];
  tr_twiddle<1, R>(v, tw, j);
  tr_dft<R, 1>(v);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float2 t = cmulc(s[r], cscale(v[r], scale));
    if (ok) sum[r] = cadd(sum[r], t);
  }
}

template <int R>
__device__ __forceinline__ void combine_put(const float2 (&sum)[16], float2* d, int j, int nb, int n) {
#pragma unroll
  for (int r = 0; r < R; ++r) d[centred<R>(j, r, nb, n)] = sum[r];
}

// One thread per butterfly of either pass: blockDim.x >= lines max(r0, r1).
__global__ __launch_bounds__(TR_NT, 1) void fft_combine_kernel(FftAxisArgs a, const float2* __restrict__ S, int J,
                                                               float2* __restrict__ out) {
  extern __shared__ float2 lds[];
  const int n = (int)a.n, T = a.lines, r0 = (int)a.tr_r0.d, r1 = (int)a.tr_r1.d, RP = r1 | 1, LL = r0 * RP;
  float2* tw = lds + T * LL;
  for (int i = threadIdx.x; i < n; i += blockDim.x) tw[i] = a.twiddle[i];
  const int64_t row = blockIdx.x, cs = (int64_t)a.outer_per_coil * n;
  int l0, j0, l1, j1;
  tr_coords(a, threadIdx.x, a.tr_r1, l0, j0);  // pass 0: r1 butterflies of radix r0 per line
  tr_coords(a, threadIdx.x, a.tr_r0, l1, j1);  // pass 1: r0 butterflies of radix r1
  const bool on0 = l0 < T, on1 = l1 < T;
  l0 = on0 ? l0 : 0;
  l1 = on1 ? l1 : 0;
  const float scale = rsqrtf((float)n);
  float2 in[16], s[16], sum[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) sum[r] = make_float2(0.f, 0.f);
  const float2 *src = a.src + row * n, *maps = S + row * n;
#define CB_LOAD(R) case R: combine_load<R>(in, src + min(l0, J - 1) * cs, j0, r1, n); break;
  switch (r0) { TR_SMALL(CB_LOAD) default: break; }
#undef CB_LOAD
  for (int c0 = 0; c0 < J; c0 += T) {
    if (c0 > 0) __syncthreads();  // the tile before is used up
    if (on0) {
#define CB_P0(R) case R: combine_pass0<R>(in, lds + l0 * LL + j0, RP); break;
      switch (r0) { TR_SMALL(CB_P0) default: break; }
#undef CB_P0
    }
#define CB_LOAD(R) case R: combine_load<R>(s, maps + min(c0 + l1, J - 1) * cs, j1, r0, n); break;
    switch (r1) { TR_SMALL(CB_LOAD) default: break; }
#undef CB_LOAD
#define CB_LOAD(R) case R: combine_load<R>(in, src + min(c0 + T + l0, J - 1) * cs, j0, r1, n); break;
    switch (r0) { TR_SMALL(CB_LOAD) default: break; }
#undef CB_LOAD
    __syncthreads();
#define CB_P1(R) case R: combine_pass1<R>(sum, s, lds + l1 * LL + j1 * RP, tw, j1, scale, on1 && c0 + l1 < J); break;
    switch (r1) { TR_SMALL(CB_P1) default: break; }
#undef CB_P1
  }
  __syncthreads();
  if (on1) {  // the lines' sums as rows of n (n <= r0 (r1 | 1))
#define CB_PUT(R) case R: combine_put<R>(sum, lds + l1 * n, j1, r0, n); break;
    switch (r1) { TR_SMALL(CB_PUT) default: break; }
#undef CB_PUT
  }
  __syncthreads();
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    float2 t = lds[k];
    for (int l = 1; l < T; ++l) t = cadd(t, lds[l * n + k]);
    out[row * n + k] = t;
  }
}

}  // namespace

// Two radices of at most 16, and rows enough for a workgroup on most compute units: with 64 rows
// the separate passes spread the coils over the chip instead.  With many rows they win too: a
// workgroup here runs at one wave per SIMD and holds few threads where the row is short.  Normal
// operator, this / separate: 256 rows of 256 at 32 coils 41.2 / 49.8 us, of 16 at 2 coils 15.3 / 17.4;
// 1024 rows of 90 at 32 coils 64.2 / 56.6, of 128 at 8 coils 39.2 / 39.5; 8192 rows of 128 at 8 coils 172 /
// 150, of 4 at 2 coils 39.8 / 24.6; 160000 rows of 4 at 2 coils 464 / 70.
// With few coils the launch that is saved carries the pass a little further: 640 rows of 64 at 4 coils
// 21.8 / 24.3, 900 of 240 at 8 coils 49.8 / 53.8.
bool fft_combine_supported(int64_t n, int64_t rows, int J) {
  int r0, r1;
  return rows >= 128 && rows <= (J <= 8 ? 960 : 512) && fft_tr_radices(n, r0, r1) && r0 <= 16 && r1 <= 16;
}

hipError_t fft_combine_launch(const float2* src, const float2* S, int64_t n, int64_t rows, int J, const float2* twiddle,
                              float2* out, hipStream_t st) {
  int r0, r1;
  if (!fft_combine_supported(n, rows, J) || !fft_tr_radices(n, r0, r1) || J < 1) return hipErrorInvalidValue;
  FftAxisArgs a;
  std::memset(&a, 0, sizeof(a));
  a.src = src;
  a.n = n;
  a.inner = 1;
  a.outer_per_coil = rows;
  a.twiddle = twiddle;
  a.tr_r0 = fast_div((uint32_t)r0);
  a.tr_r1 = fast_div((uint32_t)r1);
  const int nb = r0 > r1 ? r0 : r1;
  int T = 1;  // coils per tile: one butterfly per thread, no more than the coils need
  while (2 * T * nb <= TR_NT && T < J) T *= 2;
  a.lines = T;
  const int threads = (T * nb + 63) / 64 * 64;
  const size_t lds = ((size_t)T * r0 * (r1 | 1) + n) * sizeof(float2);
  hipLaunchKernelGGL(fft_combine_kernel, dim3((unsigned)rows), dim3(threads), lds, st, a, S, J, out);
  return hipGetLastError();
}

}  // namespace mx
