// Dense basis apply in FP32 (stream_apply.h).
#include "stream_apply.h"

namespace mx {

hipError_t stream_maps_fp32(const ApplyCall& a, hipStream_t st) { return dispatch<0, false>(a, st); }

hipError_t stream_apply_launch(const float2* B, int64_t N, int64_t K, const float2* c, int J, int precision, float2* S,
                               hipStream_t st) {
  if (N <= 0 || K <= 0 || J <= 0) return hipSuccess;
  const ApplyCall a{B, N, (int)K, c, J, S, nullptr, 1.f, nullptr, nullptr, 8};
  return precision == 1 ? stream_maps_bf16(a, st) : stream_maps_fp32(a, st);
}

hipError_t stream_gx_launch(const float2* B, int64_t N, int64_t K, const float2* c, int J, int precision,
                            const float2* g, float alpha, const float* alpha_dev, float2* gx, hipStream_t st) {
  if (N <= 0 || K <= 0 || J <= 0) return hipSuccess;
  const ApplyCall a{B, N, (int)K, c, J, nullptr, g, alpha, alpha_dev, gx, 8};
  return precision == 1 ? stream_gx_bf16(a, st) : stream_gx_fp32(a, st);
}

}  // namespace mx
