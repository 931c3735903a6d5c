// gemm_dl instantiations: 256x256 tiles: problems with enough of them to fill the chip.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_256(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<bf16_t, 256, 256, false>(g, akc, bkc, epi, s);
}

}  // namespace atom
