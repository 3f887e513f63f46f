// Two-radix DFT passes of an image, radices up to 16 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr16_launch(const FftLaunch& l, hipStream_t st) {
  return l.variant >= TR_GRID_FIRST && l.variant <= TR_GRID_LAST ? fft_tr16_grid(l, st) : tr_launch_one<false, false>(l, st);
}

}  // namespace mx
