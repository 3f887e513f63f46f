// Two-radix DFT passes of an image, radices up to 32 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr32_launch(const FftLaunch& l, hipStream_t st) {
  return l.variant >= TR_GRID_FIRST && l.variant <= TR_GRID_LAST ? fft_tr32_grid(l, st) : tr_launch_one<true, false>(l, st);
}

}  // namespace mx
