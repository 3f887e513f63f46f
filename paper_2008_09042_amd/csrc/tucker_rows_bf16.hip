// Tucker products next to the coil images in BF16-split (tucker_rows.h).
#include "tucker_rows.h"

namespace mx {

hipError_t tucker_maps_bf16(const RowsArgs& r, hipStream_t st) { return maps_by_rank<1>(r, st); }
hipError_t tucker_images_bf16(const RowsArgs& r, hipStream_t st) { return images_by_rank<1>(r, st); }
hipError_t tucker_mode1_bf16(const TuckerRows& a, const float2* Q3, float2* Q2, hipStream_t st) {
  return mode1_by_rank<1>(a, Q3, Q2, st);
}

}  // namespace mx
