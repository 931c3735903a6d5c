// gemm_dl instantiations: 128x128 tiles, two workgroups per CU.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_128(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<bf16_t, 128, 128, false>(g, akc, bkc, epi, s);
}

}  // namespace atom
