// gemm_dl instantiations: 256x128 tiles, between 256x256 and 128x128.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_256x128(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<bf16_t, 256, 128, true>(g, akc, bkc, epi, s);
}

}  // namespace atom
