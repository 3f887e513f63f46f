// Two-radix DFT passes with radices up to 32 (fft_tr.h).
#include "fft_tr.h"

namespace mx {

hipError_t fft_tr32_launch(const FftLaunch& l, hipStream_t st) { return tr_launch_one<true>(l, st); }

hipError_t fft_tr32_multi(int variant, int threads, size_t lds, const FftMulti& m, hipStream_t st) {
  return tr_launch_many<true>(variant, threads, lds, m, st);
}

}  // namespace mx
