// V-Major selection as the paper states it (Section III-D): a per-token scalar (L1 distance between the
// token's current and cached value vector), the fraction r with the smallest distance stays cached, the other
// tokens are active; r comes from the time-varying cache schedule (warm-up, linear ramp, periodic full update).
//
//   token_metric_kernel -- one wavefront per token streams the token's value vector from both tensors once
//                          (HBM-bound), fp32 sum of |cur - prev| per lane, wavefront tree reduction;
//   topk_kernel         -- one workgroup per segment (a logical rank's tokens), keys in registers: the K-th largest
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
constexpr int kTopkUnroll = 8;                // metric values a lane has in flight where the keys are not kept
constexpr int kTopkBinBits = 11;              // bins of a pass: two per lane

// Exclusive prefix sum of `v` over the workgroup in thread order; `total` gets the workgroup's sum.  (The caller has a barrier
// between two calls: wave_tot is read to the end.)
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* wave_tot, uint32_t& total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off, 64);
        if (lane >= (uint32_t)off) incl += up;
    }
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

// One workgroup per segment (a logical rank's tokens); wavefront w owns a run of `steps` 64 neighbouring tokens.  STEPS > 0: a lane
// keeps the keys of its (at most STEPS) tokens in registers after one read of the metric; 0: every pass reads the metric again
// (L2-resident), kTopkUnroll values in flight.
// One workgroup's chain of passes: bound by latency (the trip to memory, barriers, LDS atomics on one address), not by bytes.
// So the metric is asked for in one burst, and the bins of a pass divide the range the keys really have -- smallest to largest
// key first, then the bin that holds the K-th largest -- into 2048: digits at fixed places put most keys of a metric, which share
// sign and exponent, on one address, whose atomics are served one at a time.  Three passes at most; a pass whose bin is taken whole
// is the last.  (12480 tokens, a metric of two clusters: the token update around it 142.8 us with four passes over fixed
// bytes, 133.5 so with the keys in LDS, eight loads in flight; 130.8 with the keys in registers and all loads in flight.  29520
// tokens 229.4 -> 224.4; 43632 tokens, not kept, 349.5 -> 348.0.)
// The list is written by 64 neighbouring tokens at a time (ballots).
template <int STEPS>
__global__ void __launch_bounds__(kTopkThreads) topk_kernel(const float* __restrict__ metric, uint32_t N, uint32_t K,
                                                            int32_t* __restrict__ idx, int32_t* __restrict__ n_active,
                                                            uint32_t id_stride) {
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
    const uint32_t steps = (N + kTopkThreads - 1) / kTopkThreads, run = wave * steps * 64u;
    // f(s, key) for the keys of this lane's tokens run + 64 s + lane; beyond the segment's end the key is 0, which no metric has
    // (the smallest is that of -infinity) and which lies outside every range of real keys
    constexpr int kGroup = STEPS ? STEPS : kTopkUnroll;
    uint32_t kept[kGroup];
    auto load = [&](uint32_t s0) __attribute__((always_inline)) {
        float m[kGroup];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) m[k] = metric[min(run + 64u * (s0 + k) + lane, N - 1u)];
#pragma unroll
        for (int k = 0; k < kGroup; ++k) {
            const uint32_t s = s0 + k;
            kept[k] = s < steps && run + 64u * s + lane < N ? metric_key(m[k]) : 0u;
        }
    };
    auto for_keys = [&](auto f) __attribute__((always_inline)) {
        for (uint32_t s0 = 0; s0 < (STEPS ? 1u : steps); s0 += kGroup) {
            if (!STEPS) load(s0);
#pragma unroll
            for (int k = 0; k < kGroup; ++k)
                if (s0 + k < steps) f(s0 + k, kept[k]);
        }
    };
    if (STEPS) load(0);
    // ---- the keys' range
    uint32_t low = 0xFFFFFFFFu, high = 0;
    for_keys([&](uint32_t, uint32_t key) __attribute__((always_inline)) {
        low = min(low, key ? key : 0xFFFFFFFFu);
        high = max(high, key);
    });
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
    // ---- the K-th largest key: in [low, low + range], the `remaining`-th largest there
    uint32_t range = high - low, remaining = K;
    bool whole;      // every key of the last bin is taken
    for (;;) {
        const int bits = range ? 32 - __clz((int)range) : 0, shift = bits > kTopkBinBits ? bits - kTopkBinBits : 0;
        for_keys([&](uint32_t, uint32_t key) __attribute__((always_inline)) {
            const uint32_t off = key - low;
            if (off <= range) atomicAdd(&hist[off >> shift], 1u);
        });
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
        range = min((1u << shift) - 1u, 0xFFFFFFFFu - low);      // (not past the largest key, to the key 0 of no token)
        remaining = s_remaining;
        whole = remaining == s_count;
        if (whole || shift == 0) break;
    }
    // ---- compaction in index order: take keys above `low`, and equal to it while there is room (`whole`: from `low` up)
    auto look = [&](uint32_t key, uint64_t& above, uint64_t& equal) __attribute__((always_inline)) {
        above = __ballot(key > low || (whole && key == low));
        equal = __ballot(!whole && key == low);
    };
    uint32_t n_above = 0, n_equal = 0;
    for_keys([&](uint32_t, uint32_t key) __attribute__((always_inline)) {
        uint64_t above, equal;
        look(key, above, equal);
        n_above += __popcll(above);
        n_equal += __popcll(equal);
    });
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
    const uint64_t before = (1ull << lane) - 1ull;
    for_keys([&](uint32_t s, uint32_t key) __attribute__((always_inline)) {
        uint64_t above, equal;
        look(key, above, equal);
        const uint32_t equal_here = equal_before + __popcll(equal & before);
        const bool take_equal = ((equal >> lane) & 1u) && equal_here < rest;
        const uint64_t taken = above | __ballot(take_equal);
        if ((taken >> lane) & 1u) idx[pos + __popcll(taken & before)] = (int32_t)(id_base + run + 64u * s + lane);
        pos += __popcll(taken);
        equal_before += __popcll(equal);
    });
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
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_seg), dim3(kTopkThreads), 0, as_stream(stream), metric, (uint32_t)N, (uint32_t)n_keep, active_idx,
                           n_active, global_ids ? (uint32_t)N : 0u);
    };
    // keys in registers up to 32 per lane: 16 wavefronts of a workgroup leave each 128 registers
    if (N <= 4 * kTopkThreads) launch(topk_kernel<4>);
    else if (N <= 16 * kTopkThreads) launch(topk_kernel<16>);
    else if (N <= 32 * kTopkThreads) launch(topk_kernel<32>);
    else launch(topk_kernel<0>);
    return check_launch("topk_kernel");
}

extern "C" int32_t cocodiff_cache_active_count(int32_t step, int32_t n_steps, int32_t warmup, int32_t sync_every,
                                               int32_t n_tokens) {
    if (n_tokens <= 0 || step < 1 || n_steps < 1 || warmup < 0) return -1;
    if (step <= warmup || n_steps <= warmup || (sync_every > 0 && step % sync_every == 0)) return n_tokens;   // full exchange
    const int64_t cached = (int64_t)n_tokens * (step - warmup) / (n_steps - warmup);   // floor(r * n_tokens), r = linear ramp
    return (int32_t)(n_tokens - (cached > n_tokens ? n_tokens : cached));
}
