// gemm_dl instantiations: fp32 tiles.
#include "gemm_dl.h"

namespace atom {

hipError_t gemm_dl_f32_64(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<float, 64, 64, false>(g, akc, bkc, epi, s);
}
hipError_t gemm_dl_f32_32(const GemmArgs& g, bool akc, bool bkc, int epi, hipStream_t s) {
  return dl::launch<float, 32, 32, false>(g, akc, bkc, epi, s);
}

}  // namespace atom
