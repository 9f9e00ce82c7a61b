// The projection's main kernel writing both, Q and K normalised and rotated by any table.
#include "gemm_kernel.h"

namespace cocodiff {

#define ENTRY(NI, NJ) (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_FUSED_ANY>,
const void* const kFusedAnyKernels[] = {COCODIFF_FUSED_TILES(ENTRY) COCODIFF_FUSED_LONG_TILES(ENTRY)};
#undef ENTRY

}  // namespace cocodiff
