// Tucker products of the general 3D path around the coil images (tucker_rows.h).
#pragma once

#include "common.h"

namespace mx {

struct TuckerRows {
  int64_t n0, n1, n2, r0, r1, r2;
  int J;
  const float2 *U1, *U2;  // [n1][r1], [n2][r2]
  int precision;
};

bool tucker_rows_supported(int64_t n0, int64_t n1, int64_t n2, int64_t r1, int64_t r2, int precision);
// Whether tucker_images_launch is also the way to gx, rather than maps in memory and their combination.
bool tucker_images_gx_fits(int64_t n0, int64_t n1, int J, int precision);
// Stacks of coil images are 16-byte aligned.
// S [J][n0][n1][n2] = T2 [J][n0][r1][r2] x_2 U1 x_3 U2
hipError_t tucker_maps_launch(const TuckerRows& a, const float2* T2, float2* S, hipStream_t st);
// From the coil images g [J][n0][n1][n2]: gx = s sum_j conj(S_j) (.) g_j, s = alpha (* alpha_dev),
// with S formed from T2 in registers, and Q3 [J][n0][n1][r2] = h x_3 U2^H for h = conj(x) (.) g
// (h = g without x).  gx or Q3 may be null; x and T2 are not read where they are not needed.
hipError_t tucker_images_launch(const TuckerRows& a, const float2* T2, const float2* x, const float2* g, float alpha,
                                const float* alpha_dev, float2* gx, float2* Q3, hipStream_t st);
// Q2 [J][n0][r1][r2] = Q3 x_2 U1^H
hipError_t tucker_mode1_adjoint_launch(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st);

}  // namespace mx
