// Image gradient of a dense basis in FP32 (stream_apply.h).
#include "stream_apply.h"

namespace mx {

hipError_t stream_gx_fp32(const ApplyCall& a, hipStream_t st) { return dispatch<0, true>(a, st); }

}  // namespace mx
