// Two-radix DFT passes of a gridding window, radices up to 32 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr32_grid(const FftLaunch& l, hipStream_t st) { return tr_launch_one<true, true>(l, st); }

}  // namespace mx
