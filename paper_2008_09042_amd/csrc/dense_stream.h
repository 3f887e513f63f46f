// Dense basis products as streams of the basis (stream_apply.h, stream_adjoint.h).
#pragma once

#include "common.h"

namespace mx {

// S [J][N] = B [N][K] c^T for c [J][K].
hipError_t stream_apply_launch(const float2* B, int64_t N, int64_t K, const float2* c, int J, int precision, float2* S,
                               hipStream_t st);
// gx[n] = s sum_j conj((B c_j)[n]) g[j][n], s = alpha (* alpha_dev): the maps are formed and
// consumed in registers.
hipError_t stream_gx_launch(const float2* B, int64_t N, int64_t K, const float2* c, int J, int precision,
                            const float2* g, float alpha, const float* alpha_dev, float2* gx, hipStream_t st);
// c [J][K] = s B^H h, with h = conj(x) (.) g formed on the way when x [N] is given and h = g
// otherwise; ws holds stream_adjoint_bytes (the row chunks' partials, summed in a fixed order; at
// most max_chunks of them, 0: no limit).
size_t stream_adjoint_bytes(int64_t N, int64_t K, int J, int max_chunks);
hipError_t stream_adjoint_launch(const float2* B, int64_t N, int64_t K, const float2* g, const float2* x, int J,
                                 int precision, float alpha, const float* alpha_dev, void* ws, int max_chunks,
                                 float2* c, hipStream_t st);

}  // namespace mx
