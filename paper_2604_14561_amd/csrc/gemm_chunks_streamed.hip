// The projection's main kernel writing the exchange-buffer chunks, streamed past the caches.
#include "gemm_kernel.h"

namespace cocodiff {

#define ENTRY(NI, NJ) (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_CHUNKS_STREAMED>,
const void* const kChunkStreamedKernels[] = {COCODIFF_PLAIN_TILES(ENTRY) COCODIFF_PLAIN_LONG_TILES(ENTRY)};
#undef ENTRY

}  // namespace cocodiff
