// Z = (M + G) Q   (PowerIter1, first product): A = fused sum read along k = n, B = Q read across k.
#include "gemm_dispatch.hpp"
namespace dion {
hipError_t gemm_k1(int variant, bool bf16, bool gbf16, GemmArgs g, int batch, hipStream_t s) {
  return dispatch_types<CfgBig, CfgSmall, PRODUCT_VARIANTS, SRC_SUM_KC, SRC_F32_KS, EPI_STORE, false>(variant, bf16, gbf16, g, batch, s);
}
}  // namespace dion
