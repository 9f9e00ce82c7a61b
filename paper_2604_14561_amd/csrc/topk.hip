// V-Major selection as the paper states it (Section III-D): a per-token scalar (L1 distance between the
// token's current and cached value vector), the fraction r with the smallest distance stays cached, the other
// tokens are active; r comes from the time-varying cache schedule (warm-up, linear ramp, periodic full update).
//
//   token_metric_kernel -- one wavefront per token streams the token's value vector from both tensors once
//                          (HBM-bound), fp32 sum of |cur - prev| per lane, wavefront tree reduction;
//   topk_kernel         -- one workgroup per segment (a logical rank's tokens), keys cached in LDS: the K-th largest
//                          key by histograms over a range of keys that each pass narrows, then an
//                          index-ordered compaction that takes every token above the threshold and the
//                          lowest-indexed tokens equal to it until K are taken.
#include "internal.h"

namespace cocodiff {

constexpr int kMetricWaves = 4;
constexpr int kMetricUnroll = 6;

// metric[n] = sum over slabs s and w of |cur[s][n][w] - prev[s][n][w]|
template <bool NT_CUR, bool NT_PREV>
__global__ void __launch_bounds__(64 * kMetricWaves) token_metric_kernel(const vec16* __restrict__ cur, const vec16* __restrict__ prev,
                                                                         float* __restrict__ metric, uint32_t S, uint32_t N, uint32_t W8) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t n = blockIdx.x * kMetricWaves + (threadIdx.x >> 6);
    if (n >= N) return;
    const uint32_t total = S * W8;
    float acc = 0.f;
    for (uint32_t g0 = lane; g0 < total; g0 += 64 * kMetricUnroll) {
        vec16 c[kMetricUnroll], p[kMetricUnroll];
#pragma unroll
        for (int k = 0; k < kMetricUnroll; ++k) {
            const uint32_t g = g0 + 64 * k;
            if (g < total) {
                const uint32_t s = g / W8, v = g - s * W8;
                const uint64_t at = ((uint64_t)s * N + n) * W8 + v;
                c[k] = ld_vec<NT_CUR>(cur + at);
                p[k] = ld_vec<NT_PREV>(prev + at);
            }
        }
#pragma unroll
        for (int k = 0; k < kMetricUnroll; ++k) {
            if (g0 + 64 * k < total) {
                const uint32_t cw[4] = {c[k].x, c[k].y, c[k].z, c[k].w};
                const uint32_t pw[4] = {p[k].x, p[k].y, p[k].z, p[k].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc += fabsf(bf16_lo(cw[i]) - bf16_lo(pw[i]));
                    acc += fabsf(bf16_hi(cw[i]) - bf16_hi(pw[i]));
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) metric[n] = acc;
}

// Order-preserving key: larger metric <-> larger key; every NaN maps to the largest key; -0 and +0 share one.
__device__ __forceinline__ uint32_t metric_key(float m) {
    if (m != m) return 0xFFFFFFFFu;
    const uint32_t b = m == 0.f ? 0u : __float_as_uint(m);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kTopkUnroll = 8;                // metric values a lane has in flight
constexpr int kTopkBinBits = 11;              // bins of a pass: two per lane
constexpr uint32_t kTopkCachedKeys = 32768;   // keys of one segment kept in LDS (128 KB) when they fit

// Exclusive prefix sum of `v` over the workgroup in thread order; `total` gets the workgroup's sum.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* wave_tot, uint32_t& total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off, 64);
        if (lane >= (uint32_t)off) incl += up;
    }
    __syncthreads();                               // wave_tot may still be read from the previous call
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kTopkWaves; ++w) {
        const uint32_t c = wave_tot[w];
        before += (uint32_t)w < wave ? c : 0u;
        tot += c;
    }
    total = tot;
    return before + incl - v;
}

// One workgroup per segment (a logical rank's tokens).  CACHED: the segment's keys sit in LDS after one read of
// the metric; otherwise every pass reads the metric again (L2-resident).
// One workgroup's chain of passes: bound by latency (barriers, LDS atomics on one address), not by bytes.  So the bins of a
// pass divide the range the keys really have -- smallest to largest key first, then the bin that holds the K-th largest --
// into 2048: digits at fixed places put most keys of a metric, which share sign and exponent, on one address, whose atomics
// are served one at a time.  Three passes at most; a pass whose bin is taken whole is the last.  (12480 tokens, a metric of two
// clusters: the token update around it 142.8 us with four passes over fixed bytes, 134.1 so.)
// The list is written by 64 neighbouring tokens at a time (ballots), each wavefront its own run of them.
template <bool CACHED>
__global__ void __launch_bounds__(kTopkThreads) topk_kernel(const float* __restrict__ metric, uint32_t N, uint32_t K,
                                                            int32_t* __restrict__ idx, int32_t* __restrict__ n_active,
                                                            uint32_t id_stride) {
    extern __shared__ uint32_t s_keys[];
    constexpr uint32_t kBins = 1u << kTopkBinBits;
    static_assert(kBins == 2 * kTopkThreads, "two bins per lane");
    __shared__ __align__(8) uint32_t hist[kBins];
    __shared__ uint32_t wave_tot[kTopkWaves], wave_min[kTopkWaves], wave_max[kTopkWaves];
    __shared__ uint32_t s_bin, s_remaining, s_count;
    metric += (size_t)blockIdx.x * N;
    idx += (size_t)blockIdx.x * N;
    const uint32_t id_base = blockIdx.x * id_stride;   // 0: ids local to the segment; N: ids in the whole metric array
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) n_active[blockIdx.x] = (int32_t)K;
    if (K == 0) return;
    // ---- the keys' range
    uint32_t low = 0xFFFFFFFFu, high = 0;
    for (uint32_t n0 = threadIdx.x; n0 < N; n0 += kTopkUnroll * kTopkThreads) {
        float m[kTopkUnroll];
#pragma unroll
        for (int k = 0; k < kTopkUnroll; ++k) m[k] = metric[min(n0 + k * kTopkThreads, N - 1u)];   // (the last one again beyond the end)
#pragma unroll
        for (int k = 0; k < kTopkUnroll; ++k) {
            const uint32_t key = metric_key(m[k]);
            low = min(low, key);
            high = max(high, key);
            if (CACHED && n0 + k * kTopkThreads < N) s_keys[n0 + k * kTopkThreads] = key;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        low = min(low, (uint32_t)__shfl_xor(low, off, 64));
        high = max(high, (uint32_t)__shfl_xor(high, off, 64));
    }
    if (lane == 0) {
        wave_min[wave] = low;
        wave_max[wave] = high;
    }
    *reinterpret_cast<uint2*>(hist + 2 * threadIdx.x) = uint2{0, 0};
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTopkWaves; ++w) {
        low = min(low, wave_min[w]);
        high = max(high, wave_max[w]);
    }
    auto key_at = [&](uint32_t n) { return CACHED ? s_keys[n] : metric_key(metric[n]); };
    // ---- the K-th largest key: in [low, low + range], the `remaining`-th largest there
    uint32_t range = high - low, remaining = K;
    bool whole;      // every key of the last bin is taken
    for (;;) {
        const int bits = range ? 32 - __clz((int)range) : 0, shift = bits > kTopkBinBits ? bits - kTopkBinBits : 0;
        for (uint32_t n = threadIdx.x; n < N; n += kTopkThreads) {
            const uint32_t off = key_at(n) - low;
            if (off <= range) atomicAdd(&hist[off >> shift], 1u);
        }
        __syncthreads();
        // bins from the top, two per lane; `above` = keys of the range in higher bins
        const uint32_t top = kBins - 1u - 2u * threadIdx.x;
        const uint2 two = *reinterpret_cast<const uint2*>(hist + top - 1u);
        uint32_t in_play, above = block_scan(two.x + two.y, wave_tot, in_play);
        *reinterpret_cast<uint2*>(hist + top - 1u) = uint2{0, 0};      // for the next pass
#pragma unroll
        for (uint32_t i = 0; i < 2; ++i) {
            const uint32_t count = i == 0 ? two.y : two.x;
            if (above < remaining && above + count >= remaining) {      // exactly one bin: 1 <= remaining <= in_play
                s_bin = top - i;
                s_remaining = remaining - above;       // how many keys of this bin to take
                s_count = count;
            }
            above += count;
        }
        __syncthreads();
        low += s_bin << shift;
        range = (1u << shift) - 1u;
        remaining = s_remaining;
        whole = remaining == s_count;
        if (whole || shift == 0) break;
    }
    // ---- compaction in index order: take keys above `low`, and equal to it while there is room (`whole`: from `low` up);
    // wavefront w owns a run of `steps` 64 tokens
    const uint32_t steps = (N + kTopkThreads - 1) / kTopkThreads, run = wave * steps * 64u;
    auto look = [&](uint32_t s, uint64_t& above, uint64_t& equal) __attribute__((always_inline)) {
        const uint32_t n = run + 64u * s + lane, key = n < N ? key_at(n) : 0u;
        above = __ballot(n < N && (key > low || (whole && key == low)));
        equal = __ballot(n < N && !whole && key == low);
    };
    uint32_t n_above = 0, n_equal = 0;
    for (uint32_t s = 0; s < steps; ++s) {
        uint64_t above, equal;
        look(s, above, equal);
        n_above += __popcll(above);
        n_equal += __popcll(equal);
    }
    if (lane == 0) {
        wave_min[wave] = n_above;
        wave_max[wave] = n_equal;
    }
    __syncthreads();
    uint32_t pos = 0, equal_before = 0;
    for (uint32_t w = 0; w < wave; ++w) {
        pos += wave_min[w];
        equal_before += wave_max[w];
    }
    const uint32_t rest = whole ? 0u : remaining;      // equal keys taken in all, the lowest-indexed ones
    pos += min(equal_before, rest);
    for (uint32_t s = 0; s < steps; ++s) {
        uint64_t above, equal;
        look(s, above, equal);
        const uint64_t before = (1ull << lane) - 1ull;
        const uint32_t equal_here = equal_before + __popcll(equal & before);
        const bool take_equal = ((equal >> lane) & 1u) && equal_here < rest;
        const uint64_t taken = above | __ballot(take_equal);
        if ((taken >> lane) & 1u) idx[pos + __popcll(taken & before)] = (int32_t)(id_base + run + 64u * s + lane);
        pos += __popcll(taken);
        equal_before += __popcll(equal);
    }
}

}  // namespace cocodiff

using namespace cocodiff;

extern "C" int cocodiff_vmajor_token_metric(int32_t S, int32_t N, int32_t W, const cocodiff_bf16* v_cur,
                                            const cocodiff_bf16* v_prev, float* metric, void* stream) {
    if (S <= 0 || N <= 0 || W <= 0) return fail(COCODIFF_ERR_SHAPE, "token_metric: S, N, W must be positive");
    if (W % 8) return fail(COCODIFF_ERR_SHAPE, "token_metric: W (%d) must be a multiple of 8", W);
    if ((int64_t)S * (W / 8) >= ((int64_t)1 << 31)) return fail(COCODIFF_ERR_SHAPE, "token_metric: value vector too long");
    if (!v_cur || !v_prev || !metric) return fail(COCODIFF_ERR_NULL, "token_metric: NULL pointer");
    if (!aligned16(v_cur) || !aligned16(v_prev)) return fail(COCODIFF_ERR_ALIGN, "token_metric: tensors must be 16-byte aligned");
    const dim3 grid(((uint32_t)N + kMetricWaves - 1) / kMetricWaves), block(64 * kMetricWaves);
    const size_t touched = (size_t)S * N * W * 4;
    with_policy(stream_loads(touched), stream_loads_once(touched), [&](auto C, auto Pv) {
        hipLaunchKernelGGL((token_metric_kernel<decltype(C)::value, decltype(Pv)::value>), grid, block, 0, as_stream(stream),
                           (const vec16*)v_cur, (const vec16*)v_prev, metric, (uint32_t)S, (uint32_t)N, (uint32_t)(W / 8));
    });
    return check_launch("token_metric_kernel");
}

extern "C" int cocodiff_vmajor_topk(int32_t n_seg, int32_t N, const float* metric, int32_t n_keep, int32_t global_ids,
                                    int32_t* active_idx, int32_t* n_active, void* stream) {
    if (n_seg <= 0 || N <= 0) return fail(COCODIFF_ERR_SHAPE, "topk: n_seg and N must be positive");
    if ((int64_t)n_seg * N >= ((int64_t)1 << 31)) return fail(COCODIFF_ERR_SHAPE, "topk: n_seg * N must be below 2^31");
    if (n_keep < 0 || n_keep > N) return fail(COCODIFF_ERR_SHAPE, "topk: n_keep (%d) must be in [0, N = %d]", n_keep, N);
    if (!metric || !active_idx || !n_active) return fail(COCODIFF_ERR_NULL, "topk: NULL pointer");
    if ((uint32_t)N <= kTopkCachedKeys) {
        static int lds_ok = [] {
            return (int)hipFuncSetAttribute((const void*)topk_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)(kTopkCachedKeys * sizeof(uint32_t)));
        }();
        if (lds_ok != (int)hipSuccess) return fail(COCODIFF_ERR_HIP, "topk: cannot raise the kernel's LDS limit");
        hipLaunchKernelGGL(topk_kernel<true>, dim3(n_seg), dim3(kTopkThreads), (size_t)N * sizeof(uint32_t), as_stream(stream),
                           metric, (uint32_t)N, (uint32_t)n_keep, active_idx, n_active, global_ids ? (uint32_t)N : 0u);
    } else {
        hipLaunchKernelGGL(topk_kernel<false>, dim3(n_seg), dim3(kTopkThreads), 0, as_stream(stream), metric, (uint32_t)N,
                           (uint32_t)n_keep, active_idx, n_active, global_ids ? (uint32_t)N : 0u);
    }
    return check_launch("topk_kernel");
}

extern "C" int32_t cocodiff_cache_active_count(int32_t step, int32_t n_steps, int32_t warmup, int32_t sync_every,
                                               int32_t n_tokens) {
    if (n_tokens <= 0 || step < 1 || n_steps < 1 || warmup < 0) return -1;
    if (step <= warmup || n_steps <= warmup || (sync_every > 0 && step % sync_every == 0)) return n_tokens;   // full exchange
    const int64_t cached = (int64_t)n_tokens * (step - warmup) / (n_steps - warmup);   // floor(r * n_tokens), r = linear ramp
    return (int32_t)(n_tokens - (cached > n_tokens ? n_tokens : cached));
}
