// Two-radix DFT passes of several slices, radices up to 32 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr32_multi(int variant, int threads, size_t lds, const FftMulti& m, hipStream_t st) {
  return tr_launch_many<true>(variant, threads, lds, m, st);
}

}  // namespace mx
