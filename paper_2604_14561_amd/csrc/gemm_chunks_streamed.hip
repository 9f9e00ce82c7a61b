// The projection's main kernel writing the exchange-buffer chunks, streamed past the caches in whole lines: tiles whose wavefronts have
// their groups of 32 features in pairs, 256 and 128 features wide.  The others have no such kernel.
#include "gemm_kernel.h"

namespace cocodiff {

#define ENTRY(NI, NJ) NI % 4 ? nullptr : (const void*)qkv_gemm_direct_kernel<NI % 4 ? 8 : NI, NI % 4 ? 8 : NJ, OUT_CHUNKS_STREAMED>,
const void* const kChunkStreamedKernels[] = {COCODIFF_PLAIN_TILES(ENTRY) COCODIFF_PLAIN_LONG_TILES(ENTRY)};
#undef ENTRY

}  // namespace cocodiff
