// Dense basis adjoint in BF16-split (stream_adjoint.h).
#include "stream_adjoint.h"

namespace mx {

hipError_t stream_adjoint_bf16(const AdjCall& a, hipStream_t st) { return adjoint<1>(a, st); }

}  // namespace mx
