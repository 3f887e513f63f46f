// Two-radix DFT passes of a gridding window, radices up to 16 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr16_grid(const FftLaunch& l, hipStream_t st) { return tr_launch_one<false, true>(l, st); }

}  // namespace mx
