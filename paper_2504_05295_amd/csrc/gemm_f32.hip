// fp32 products of the orthonormalisation: the Gram matrix and the triangular multiply, whose sizes are the matrix' own, and
// the merges of the inverse, on blocks that are multiples of 64.
#include "gemm_dispatch.hpp"
namespace dion {
constexpr unsigned ANY_SIZE = variant_set(VAR_BIG, VAR_SMALL, VAR_SMALL_RAGGED, VAR_SMALL_CHECKED);
hipError_t gemm_f32_nt(int variant, GemmArgs g, int batch, hipStream_t s) {
  return dispatch_tiles<CfgBig, CfgSmall, ANY_SIZE, false, SRC_F32_KC, SRC_F32_KC, false, EPI_STORE, false>(variant, g, batch, s);
}
hipError_t gemm_f32_nn(int variant, GemmArgs g, int batch, hipStream_t s) {
  return dispatch_tiles<CfgBig, CfgSmall, variant_set(VAR_BIG, VAR_SMALL), false, SRC_F32_KC, SRC_F32_KS, false, EPI_STORE, false>(variant, g, batch, s);
}
hipError_t gemm_f32_tn(int variant, GemmArgs g, int batch, hipStream_t s) {
  return dispatch_tiles<CfgBig, CfgSmall, ANY_SIZE, false, SRC_F32_KS, SRC_F32_KS, false, EPI_STORE, false>(variant, g, batch, s);
}
}  // namespace dion
