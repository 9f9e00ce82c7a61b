// The projection's main kernel writing the exchange buffer's chunks.
#include "gemm_kernel.h"

namespace cocodiff {

#define ENTRY(NI, NJ) (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_CHUNKS>,
const void* const kChunkKernels[] = {COCODIFF_PLAIN_TILES(ENTRY) COCODIFF_PLAIN_LONG_TILES(ENTRY)};
#undef ENTRY

}  // namespace cocodiff
