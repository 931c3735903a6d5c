// gemm_dl instantiations: 64x64 tiles: few output tiles.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_64(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<bf16_t, 64, 64, false>(g, akc, bkc, epi, s);
}

}  // namespace atom
