// gemm_dl instantiations: 256x192 tiles, for widths that 256 columns divide badly.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_192(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<bf16_t, 256, 192, true>(g, akc, bkc, epi, s);
}

}  // namespace atom
