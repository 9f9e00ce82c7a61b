// The projection's main kernel writing both, Q and K normalised and rotated, V streamed past the caches too.
#include "gemm_kernel.h"

namespace cocodiff {

#define ENTRY(NI, NJ) (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_FUSED_STREAMED>,
const void* const kFusedStreamedKernels[] = {COCODIFF_FUSED_TILES(ENTRY) COCODIFF_FUSED_LONG_TILES(ENTRY)};
#undef ENTRY

}  // namespace cocodiff
