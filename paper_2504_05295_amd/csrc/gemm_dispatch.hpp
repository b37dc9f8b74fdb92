// Variant dispatch shared by the GEMM translation units.
#pragma once
#include "internal.hpp"

namespace dion {
// The tile variants that a product's shapes can ask for; the others are not compiled, and refused.
constexpr unsigned variant_set(int v) { return 1u << v; }
template <class... V>
constexpr unsigned variant_set(int v, V... rest) { return variant_set(v) | variant_set(rest...); }

template <class Big, class Small, unsigned SET, bool BF16, int ASRC, int BSRC, bool GBF16, int EPI, bool DUAL>
inline hipError_t dispatch_tiles(int variant, GemmArgs g, int batch, hipStream_t s) {
  if constexpr (SET & variant_set(VAR_BIG))
    if (variant == VAR_BIG) return launch_gemm<Big, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_EXACT, EDGE_EXACT>(g, batch, s);
  if constexpr (SET & variant_set(VAR_SMALL))
    if (variant == VAR_SMALL) return launch_gemm<Small, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_EXACT, EDGE_EXACT>(g, batch, s);
  if constexpr (SET & variant_set(VAR_BIG_RAGGED))
    if (variant == VAR_BIG_RAGGED) return launch_gemm<Big, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_RAGGED, EDGE_RAGGED>(g, batch, s);
  if constexpr (SET & variant_set(VAR_SMALL_RAGGED))
    if (variant == VAR_SMALL_RAGGED) return launch_gemm<Small, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_RAGGED, EDGE_RAGGED>(g, batch, s);
  if constexpr (SET & variant_set(VAR_SMALL_NARROW))
    if (variant == VAR_SMALL_NARROW) return launch_gemm<Small, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_RAGGED, EDGE_CHECKED>(g, batch, s);
  if constexpr (SET & variant_set(VAR_SMALL_CHECKED))
    if (variant == VAR_SMALL_CHECKED) return launch_gemm<Small, BF16, ASRC, BSRC, GBF16, EPI, DUAL, EDGE_CHECKED, EDGE_CHECKED>(g, batch, s);
  return hipErrorInvalidValue;
}

// the same for every operand type of the products with M + G and of the update
template <class Big, class Small, unsigned SET, int ASRC, int BSRC, int EPI, bool DUAL>
inline hipError_t dispatch_types(int variant, bool bf16, bool gbf16, GemmArgs g, int batch, hipStream_t s) {
  if (bf16)
    return gbf16 ? dispatch_tiles<Big, Small, SET, true, ASRC, BSRC, true, EPI, DUAL>(variant, g, batch, s)
                 : dispatch_tiles<Big, Small, SET, true, ASRC, BSRC, false, EPI, DUAL>(variant, g, batch, s);
  return gbf16 ? dispatch_tiles<Big, Small, SET, false, ASRC, BSRC, true, EPI, DUAL>(variant, g, batch, s)
               : dispatch_tiles<Big, Small, SET, false, ASRC, BSRC, false, EPI, DUAL>(variant, g, batch, s);
}
// (N, the rank, may be below a tile where M and K are not)
constexpr unsigned PRODUCT_VARIANTS = variant_set(VAR_BIG, VAR_SMALL, VAR_BIG_RAGGED, VAR_SMALL_RAGGED, VAR_SMALL_NARROW, VAR_SMALL_CHECKED);
// (K, the rank, is at most N: where K is a tile at least, N is)
constexpr unsigned UPDATE_VARIANTS = variant_set(VAR_BIG, VAR_SMALL, VAR_BIG_RAGGED, VAR_SMALL_RAGGED, VAR_SMALL_CHECKED);
}  // namespace dion
