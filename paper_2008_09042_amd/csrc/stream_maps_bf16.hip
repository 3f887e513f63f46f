// Dense basis apply in BF16-split (stream_apply.h).
#include "stream_apply.h"

namespace mx {

hipError_t stream_maps_bf16(const ApplyCall& a, hipStream_t st) { return dispatch<1, false>(a, st); }

}  // namespace mx
