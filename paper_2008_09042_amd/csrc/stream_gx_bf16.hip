// Image gradient of a dense basis in BF16-split (stream_apply.h).
#include "stream_apply.h"

namespace mx {

hipError_t stream_gx_bf16(const ApplyCall& a, hipStream_t st) { return dispatch<1, true>(a, st); }

}  // namespace mx
