// Tucker products next to the coil images in FP32 (tucker_rows.h), and the choice between them.
#include "tucker_rows.h"

namespace mx {

hipError_t tucker_maps_fp32(const RowsArgs& r, hipStream_t st) { return maps_by_rank<0>(r, st); }
hipError_t tucker_images_fp32(const RowsArgs& r, hipStream_t st) { return images_by_rank<0>(r, st); }
hipError_t tucker_mode1_fp32(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st) {
  return mode1_by_rank<0>(a, Q3, Q2, st);
}

namespace {

RowsArgs rows_args(const TuckerRows& a) {
  RowsArgs r{};
  r.n1 = a.n1;
  r.rows16 = (a.n1 + 15) / 16;
  r.n0 = (int)a.n0;
  r.n2 = (int)a.n2;
  r.r1 = (int)a.r1;
  r.r2 = (int)a.r2;
  r.J = a.J;
  r.jc = a.J;
  r.U1 = a.U1;
  r.U2 = a.U2;
  return r;
}

}  // namespace

bool tucker_rows_supported(int64_t n0, int64_t n1, int64_t n2, int64_t r1, int64_t r2, int precision) {
  if (n0 * n1 * n2 >= (int64_t)1 << 29) return false;  // 32-bit offsets into an image
  if (precision != 0 && precision != 1) return false;
  if (n2 < 2 || n2 > 128 || n2 % 2 || r1 < 1 || r2 < 1 || r1 > 16 * RANK_TILES || r2 > 16 * RANK_TILES) return false;
  return (n1 + 15) / 16 * ((r1 + 15) / 16) * 2048 <= 160 * 1024;  // U1's fragments (mode1_adj)
}

// With gx a wave goes through all coils of its 16 rows, one wave per SIMD (1024 on the chip).
// Where the rows leave half of them idle, the maps in memory with their combination, which
// spread the coils over the chip, are faster from a few coils on (FP32, whose products take
// longer, from fewer): the gradient in registers -> by maps, BF16-split and FP32, takes 267 -> 119
// and 351 -> 121 us at 20^3, 128 coils, ranks 8; 207 -> 120 and 338 -> 136 at 36^3, 32 coils, ranks
// 18; 133 -> 115 and 170 -> 126 at 60^3, 8 coils, ranks 20.  From 512 waves on the adjoint, which
// would have to form the maps first, is faster or even in registers (90^3, 8 coils, ranks 32:
// 142 against 172 by maps, 196 against 195; 120 x 100 x 90, 8 coils: 158 against 201, 204 against
// 229), and so it is at one or two coils everywhere (20^3: 0.91-0.95 of the time by maps).
bool tucker_images_gx_fits(int64_t n0, int64_t n1, int J, int precision) {
  return n0 * ((n1 + 15) / 16) >= 512 || J <= (precision == 1 ? 4 : 2);
}

hipError_t tucker_maps_launch(const TuckerRows& a, const float2* T2, float2* S, hipStream_t st) {
  RowsArgs r = rows_args(a);
  r.T2 = T2;
  r.S = S;
  return a.precision == 1 ? tucker_maps_bf16(r, st) : tucker_maps_fp32(r, st);
}

hipError_t tucker_images_launch(const TuckerRows& a, const float2* T2, const float2* x, const float2* g, float alpha,
                                const float* alpha_dev, float2* gx, float2* Q3, hipStream_t st) {
  RowsArgs r = rows_args(a);
  r.T2 = T2;
  r.x = x;
  r.g = g;
  r.alpha = alpha;
  r.alpha_dev = alpha_dev;
  r.gx = gx;
  r.Q3 = Q3;
  return a.precision == 1 ? tucker_images_bf16(r, st) : tucker_images_fp32(r, st);
}

hipError_t tucker_mode1_adjoint_launch(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st) {
  return a.precision == 1 ? tucker_mode1_bf16(a, Q3, Q2, st) : tucker_mode1_fp32(a, Q3, Q2, st);
}

}  // namespace mx
