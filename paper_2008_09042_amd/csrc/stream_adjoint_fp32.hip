// Dense basis adjoint in FP32 (stream_adjoint.h).
#include "stream_adjoint.h"

namespace mx {

hipError_t stream_adjoint_fp32(const AdjCall& a, hipStream_t st) { return adjoint<0>(a, st); }

size_t stream_adjoint_bytes(int64_t N, int64_t K, int J, int max_chunks) {
  if (N <= 0 || K <= 0 || J <= 0) return 0;
  return (size_t)adj_geom(N, K, J, max_chunks).nchunk * (size_t)J * (size_t)K * sizeof(float2);
}

hipError_t stream_adjoint_launch(const float2* B, int64_t N, int64_t K, const float2* g, const float2* x, int J,
                                 int precision, float alpha, const float* alpha_dev, void* ws, int max_chunks,
                                 float2* c, hipStream_t st) {
  if (N <= 0 || K <= 0 || J <= 0) return hipSuccess;
  const AdjCall a{B, N, (int)K, g, x, J, reinterpret_cast<float2*>(ws), max_chunks, alpha, alpha_dev, c};
  return precision == 1 ? stream_adjoint_bf16(a, st) : stream_adjoint_fp32(a, st);
}

}  // namespace mx
