// QKV projection (paper Section II-B): Y[n][o] = sum_k X[n][k] * W[o][k], bf16 in, fp32 accumulate on the
// gfx950 matrix cores, one RNE rounding to bf16.  The main kernel multiplies with v_mfma_f32_16x16x32_bf16: on this
// power-limited part it sustains 1.91 PFLOP/s at 0.70 pJ/flop in a register-only loop against 1.72 PFLOP/s at
// 0.77 pJ/flop for v_mfma_f32_32x32x16_bf16, for the same LDS traffic per flop (a wavefront's tile decides that).
//
// Main kernel (gemm_kernel.h; K a multiple of 64, at least three steps): K steps of 64 -- a row segment of either operand is
// one whole 128-byte line (half lines halve the L1 fill rate) -- go from global memory to LDS directly through two rings that
// turn from tile to tile of a persistent workgroup; four wavefronts, one per SIMD.  W rides the MFMA "A" side, so an
// accumulator lane holds consecutive features of one token.  Both operands are K-contiguous; LDS tiles keep rows contiguous
// and store 16-byte column c of row r at column c ^ swz(r), which makes the 128-bit fragment reads bank-conflict free.  Its
// epilogue rounds to bf16 and stores 16-byte vectors from registers: rows of [N][D], row pieces straight into their chunks of
// the exchange buffer, or row pieces of the head-parallel tensor -- or, in the fused form (tiles 128 or 256 features wide, so
// that they hold whole heads), it first RMS-normalises and rotates Q and K on the fp32 accumulators (paper Section II-B's norm
// and RoPE, one rounding in all) and writes both the chunks and the head-parallel tensor.
// The tile (tokens x features) is chosen among the built shapes by an estimate of the launch's clocks (plan_launch).
// General kernel (any K that is a multiple of 8): global -> registers -> LDS, zero-filled K tail, 256 x 256 tiles, out through
// a transpose in LDS.
#include <algorithm>
#include <initializer_list>

#include "gemm_kernel.h"

namespace cocodiff {

constexpr int BM = 256;          // tokens and features per workgroup tile of the general kernel
constexpr int kTileBytes = BM * BK * 2;                  // one operand tile of one K step of the general kernel: 32 KB
constexpr int kStageBytes = 2 * kTileBytes;              // 64 KB
constexpr int kLdsBytes = 2 * kStageBytes;               // 128 KB

// Byte offset of 16-byte column c of row r inside a [rows][64] bf16 LDS tile.
__device__ __forceinline__ uint32_t lds_off(uint32_t row, uint32_t c) { return row * 128u + ((c ^ swz(row)) << 4); }

// A wavefront's accumulators: NI feature tiles x 4 token tiles of 32 x 32.
template <int NI>
__device__ __forceinline__ void mfma_slice(f32x16 (&acc)[NI][4], const bf16x8 (&wf)[NI], const bf16x8 (&xf)[4]) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i], xf[j], acc[i][j], 0, 0, 0);
}

// Epilogue: round to bf16, transpose through this wavefront's private LDS region (ROWS token rows of COLS 16-byte
// feature columns), write whole rows.  An LDS row has CP >= COLS columns, CP a power of two; column c of row r is
// stored at column c ^ (r & (CP - 1)).
template <uint32_t COLS>
struct EpilogueRows {
    static constexpr uint32_t CP = COLS <= 4 ? 4 : COLS <= 8 ? 8 : 16;   // columns per LDS row
    static constexpr uint32_t ROWB = CP * 16;                            // bytes per LDS row
    // four consecutive features (feat a multiple of 4) of LDS row `row`
    static __device__ __forceinline__ void put4(unsigned char* ep, uint32_t row, uint32_t feat, float f0, float f1, float f2, float f3) {
        const uint32_t c16 = feat >> 3, half8 = (feat >> 2) & 1u;
        uint2 v;
        v.x = pack_bf16x2(f0, f1);
        v.y = pack_bf16x2(f2, f3);
        *reinterpret_cast<uint2*>(ep + row * ROWB + (((c16 ^ (row & (CP - 1u))) << 4) | (half8 << 3))) = v;
    }
};

// Second half of the epilogue: the wavefront reads back the rows it staged (a wavefront's LDS accesses complete in
// order: no workgroup barrier is needed) and writes them out, RPI rows per instruction.  A lane keeps its 16-byte
// feature column and walks down the rows, so every destination address is formed once (the divisions below) and then
// stepped.
// OUT_CHUNKS: the 8 features a lane writes for token n = r*Ns + m go to chunk (sender r, receiver p = feature / (Hp*d))
// of the exchange buffer Y, row m (Hp*d is a multiple of 8, so a 16-byte vector never straddles two chunks); RPI rows
// further down is RPI chunk rows further, and into sender r+1's chunk where m passes Ns (Ns >= 16 >= RPI: once at most).
// OUT_HEADS: they go to row n of head feature / d of Y = [H][N][d] (d is a multiple of 8).
template <uint32_t COLS, uint32_t ROWS, int LAYOUT>
__device__ __forceinline__ void store_rows(const unsigned char* ep, uint32_t lane, uint16_t* __restrict__ Y, size_t row0, uint32_t tok0,
                                           uint32_t feat0, uint32_t M, uint32_t D, const GemmArgs& a) {
    constexpr uint32_t CP = EpilogueRows<COLS>::CP, ROWB = EpilogueRows<COLS>::ROWB;
    constexpr uint32_t RPI = 64 / CP;            // rows per read instruction
    static_assert(RPI <= 16 && ROWS % RPI == 0, "a lane moves at most one sender's chunk further per step");
    const uint32_t c16 = lane % CP, rsub = lane / CP;
    const uint32_t feat = feat0 + c16 * 8u;
    if (c16 >= COLS || feat >= D) return;
    uint32_t tok = tok0 + rsub;
    const uint32_t n = (uint32_t)row0 + tok, v8 = feat >> 3;
    vec16* y;
    uint32_t m = 0;
    size_t step, wrap = 0;
    if (LAYOUT == OUT_CHUNKS) {
        const uint32_t r = n / a.Ns, p = v8 / a.row8, c = v8 - p * a.row8;
        m = n - r * a.Ns;
        const size_t slot = a.recv_major ? (size_t)p * a.P + r : (size_t)r * a.P + p;
        y = reinterpret_cast<vec16*>(Y) + slot * a.chunk8 + (size_t)m * a.row8 + c;
        step = (size_t)RPI * a.row8;
        wrap = a.recv_major ? 0 : (size_t)(a.P - 1u) * a.chunk8;      // slot(r + 1) - slot(r) chunks, less the Ns rows stepped over
    } else if (LAYOUT == OUT_HEADS) {
        const uint32_t h = v8 / a.d8, c = v8 - h * a.d8;
        y = reinterpret_cast<vec16*>(Y) + ((size_t)h * a.N_all + n) * a.d8 + c;
        step = (size_t)RPI * a.d8;
    } else {
        y = reinterpret_cast<vec16*>(Y + (row0 + tok) * D + feat);
        step = (size_t)RPI * (D / 8u);
    }
#pragma unroll 8
    for (uint32_t it = 0; it < ROWS / RPI; ++it) {
        if (tok < M) {
            const uint32_t row = RPI * it + rsub;
            *y = *reinterpret_cast<const vec16*>(ep + row * ROWB + ((c16 ^ (row & (CP - 1u))) << 4));
        }
        tok += RPI;
        y += step;
        if (LAYOUT == OUT_CHUNKS) {
            m += RPI;
            if (m >= a.Ns) {
                m -= a.Ns;
                y += wrap;
            }
        }
    }
}

// 32 x 32 accumulator tiles (v_mfma_f32_32x32x16_bf16): element e of lane l in tile (i, j) is feature
// 32i + 8*(e/4) + 4*(l/32) + e%4 of token 32j + l%32.
template <int NI, int NJ, int LAYOUT>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[NI][NJ], unsigned char* ep, uint32_t lane,
                                           uint16_t* __restrict__ Y, size_t row0, uint32_t tok0,
                                           uint32_t feat0, uint32_t M, uint32_t D, const GemmArgs& a) {
    const uint32_t frag_row = lane & 31u, frag_half = lane >> 5;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                EpilogueRows<NI * 4>::put4(ep, 32u * j + frag_row, 32u * i + 8u * g + 4u * frag_half, acc[i][j][4 * g + 0],
                                           acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
    store_rows<NI * 4, NJ * 32, LAYOUT>(ep, lane, Y, row0, tok0, feat0, M, D, a);
}

// ---------------------------------------------------------------------------------------------
// General path, any K that is a multiple of 8: global -> registers -> LDS, vectors beyond K are zero.
// Four wavefronts (2 x 2) of 128 x 128 outputs.
// ---------------------------------------------------------------------------------------------
constexpr int kStagedThreads = 256;
constexpr int kVecPerOperand = BM * (BK / 8) / kStagedThreads;   // 16-byte vectors per lane per operand per stage: 8

template <int LAYOUT>
__global__ void __launch_bounds__(kStagedThreads) qkv_gemm_staged_kernel(GemmArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const TileCoord tc = tile_at(a, tiles_of_block(a).first);
    const uint16_t* __restrict__ W = a.w[tc.tensor];
    const uint32_t K = (uint32_t)a.D;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t wave_f = (wave & 1u) * 128u, wave_t = (wave >> 1) * 128u;

    // lane moves vectors v = tid + 256*i of a tile: row = v/8, column = v%8
    const uint32_t ld_c = tid & 7u, ld_r = tid >> 3;
    const uint16_t* xg[kVecPerOperand];
    const uint16_t* wg[kVecPerOperand];
#pragma unroll
    for (int i = 0; i < kVecPerOperand; ++i) {
        const uint32_t r = ld_r + 32u * i;
        const uint32_t xr = min(tc.m0 + r, (uint32_t)a.M - 1u);
        const uint32_t wr = min(tc.f0 + r, (uint32_t)a.D - 1u);
        xg[i] = a.x + ((size_t)a.row_begin + xr) * K + ld_c * 8u;
        wg[i] = W + (size_t)wr * K + ld_c * 8u;
    }
    vec16 xs[kVecPerOperand], ws[kVecPerOperand];
    auto load_stage = [&](uint32_t k0) __attribute__((always_inline)) {
        const bool inside = k0 + ld_c * 8u < K;
#pragma unroll
        for (int i = 0; i < kVecPerOperand; ++i) {
            xs[i] = inside ? *reinterpret_cast<const vec16*>(xg[i] + k0) : vec16{0u, 0u, 0u, 0u};
            ws[i] = inside ? *reinterpret_cast<const vec16*>(wg[i] + k0) : vec16{0u, 0u, 0u, 0u};
        }
    };
    auto store_stage = [&](uint32_t stage) __attribute__((always_inline)) {
        unsigned char* xb = smem + stage * kStageBytes;
        unsigned char* wb = xb + kTileBytes;
#pragma unroll
        for (int i = 0; i < kVecPerOperand; ++i) {
            const uint32_t r = ld_r + 32u * i;
            *reinterpret_cast<vec16*>(xb + lds_off(r, ld_c)) = xs[i];
            *reinterpret_cast<vec16*>(wb + lds_off(r, ld_c)) = ws[i];
        }
    };

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const uint32_t n_k = (K + BK - 1) / BK;
    load_stage(0);
    store_stage(0);
    __syncthreads();
    const uint32_t frag_row = lane & 31u, frag_half = lane >> 5;
    for (uint32_t kt = 0; kt < n_k; ++kt) {
        const uint32_t cur = kt & 1u;
        if (kt + 1 < n_k) load_stage((kt + 1) * BK);
        const unsigned char* xb = smem + cur * kStageBytes;
        const unsigned char* wb = xb + kTileBytes;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 wf[4], xf[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                wf[i] = *reinterpret_cast<const bf16x8*>(wb + lds_off(wave_f + 32u * i + frag_row, 2u * kk + frag_half));
                xf[i] = *reinterpret_cast<const bf16x8*>(xb + lds_off(wave_t + 32u * i + frag_row, 2u * kk + frag_half));
            }
            mfma_slice<4>(acc, wf, xf);
        }
        if (kt + 1 < n_k) store_stage(cur ^ 1u);
        __syncthreads();
    }
    store_tile<4, 4, LAYOUT>(acc, smem + wave * (128 * 256), lane, a.y[tc.tensor], (size_t)a.row_begin, tc.m0 + wave_t,
                          tc.f0 + wave_f, (uint32_t)a.M, (uint32_t)a.D, a);
}


// A tile shape of the main kernel: tokens x features, dynamic LDS, the kernels by OutLayout.
struct TileKernel {
    int bm, bn, lds;
    int per_cu;                   // workgroups that share a compute unit
    int min_steps;                // K steps below which the shape is left out
    const void* entry[kLayouts];  // nullptr: not built
};

// K steps from which on a launch may take the shapes that lie between the others, and counts its operands more dearly (tile_clocks).
// What a shape between two others saves is operand bytes per unit (768 x 3072, Q and K fused, cold: 45.9 us with 96 x 256, 38.3 with
// 160 x 128; V plain at 2304 x 3072 48.4 with 128 x 256, 43.9 with 160 x 192): with fewer steps the start, the first trip to memory
// and the epilogue are as long as the K loop, and the estimate does not tell such shapes apart.
constexpr int kLongSteps = 16;

static const TileKernel* tile_shapes(bool whole_heads, int* count) {
#define SHAPE_FROM(STEPS, NI, NJ) {32 * NJ, 32 * NI, ring_lds_bytes(32 * NJ, 32 * NI), workgroups_per_unit(NI, NJ), STEPS, {}},
#define SHAPE(NI, NJ) SHAPE_FROM(steps_ahead(32 * NJ, 32 * NI), NI, NJ)
#define LONG_SHAPE(NI, NJ) SHAPE_FROM(kLongSteps, NI, NJ)
    static TileKernel plain[] = {COCODIFF_PLAIN_TILES(SHAPE) COCODIFF_PLAIN_LONG_TILES(LONG_SHAPE)};
    static TileKernel fused[] = {COCODIFF_FUSED_TILES(SHAPE) COCODIFF_FUSED_LONG_TILES(LONG_SHAPE)};
#undef LONG_SHAPE
#undef SHAPE
#undef SHAPE_FROM
    constexpr int n_plain = sizeof(plain) / sizeof(plain[0]), n_fused = sizeof(fused) / sizeof(fused[0]);
    static const bool filled = [] {
        for (int i = 0; i < n_plain; ++i) {
            plain[i].entry[OUT_SEQ] = kSeqKernels[i];
            plain[i].entry[OUT_CHUNKS] = kChunkKernels[i];
            plain[i].entry[OUT_HEADS] = kHeadKernels[i];
            plain[i].entry[OUT_CHUNKS_STREAMED] = kChunkStreamedKernels[i];
        }
        for (int i = 0; i < n_fused; ++i) {
            fused[i].entry[OUT_FUSED] = kFusedKernels[i];
            fused[i].entry[OUT_FUSED_ANY] = kFusedAnyKernels[i];
            fused[i].entry[OUT_FUSED_STREAMED] = kFusedStreamedKernels[i];
        }
        return true;
    }();
    (void)filled;
    *count = whole_heads ? n_fused : n_plain;
    return whole_heads ? fused : plain;
}

// Clocks of one workgroup's tile, fitted to the built shapes: a K step is 17.2 clocks per MFMA of a wavefront and 60 for its
// barrier, or the operands' way to the unit where that is longer; then the epilogue.  A round is one tile per unit also where two
// workgroups share it: they share its matrix cores and its way to L2 too.
// Operands: 37 and 40 bytes per clock and unit, fitted (some 78 GB/s).  They are for lines on chip: a launch of one round whose operands
// come from memory takes its tiles' operand bytes at 44 to 49 GB/s and unit (48 steps, 96 x 128, 160 x 128, 160 x 192 and 288 x 192
// tiles; a line counts for every unit that shares it, so all units together count more than memory delivers), much the same for
// every shape, so their order stays.
// From kLongSteps K steps on, a byte costs another 0.016 clocks where all units are busy (traffic and clock that they share),
// and the epilogue counts twice: without that, launches of many rounds took tiles of 160 x 256 and 192 x 192 for a last round a
// little fuller.  Cold inputs, three weights: 5120 x 2560 fused 199.8 us with 160 x 256, 161.6 with 224 x 256; 6144 x 3072 plain
// 287.6 with 192 x 192, 259.9 with 256 x 256; 12480 x 1536 plain 161.3 with 192 x 256, 144.7 with 256 x 256.
// Against all shapes at 768 .. 26000 tokens x 1024 .. 3072 features, one to three weights, both forms, cold inputs (110 launches):
// 0.2 % slower than the best shape on average, 6.3 % at worst; 0.8 % and 24 % with the estimate of short launches.  That one stands for
// fewer K steps: 256 .. 20736 tokens x 256 .. 3072 features (120 launches), fastest in 81 and within 3 % in 110, the others
// host-bound or plain and 4 to 8 % off but for 20736 x 256 with three weights (18.9 us for 15.9).
// On the two sides of the line, 512 .. 20736 tokens, one to three weights, both forms, cold (48 launches for each D), behind the best
// built shape on average and at worst: D 896 1.5 and 13 %, 960 1.0 and 16 % (20736 tokens, one weight, plain: 52.7 us for 45.4), 1024 0.4
// and 9.6 % (12480 tokens, three weights, plain: 80.7 for 73.7), 1088 0.2 and 4.5 %.
constexpr double kBytesPerClock = 37.0;      // of operands, per unit
static double tile_mfmas(const TileKernel& t) { return (t.bm / 32) * (t.bn / 32) * 2.0; }
static double tile_operand_bytes(const TileKernel& t) { return (t.bm + t.bn) * BK * 2.0; }
static double tile_clocks(const TileKernel& t, int32_t D, bool whole_heads, double units_busy) {
    const bool is_long = D / BK >= kLongSteps;
    const double mfmas = tile_mfmas(t), operand_bytes = tile_operand_bytes(t);
    const double step = std::max(mfmas * 17.2 + 60.0, operand_bytes / (is_long ? kBytesPerClock : 40.0)) + (is_long ? operand_bytes * 0.016 * units_busy : 0.0);
    return (D / BK) * step + (whole_heads ? 2500.0 + 100.0 * mfmas : 1500.0 + 50.0 * mfmas) * (is_long ? 2.0 : 1.0);
}

struct LaunchPlan {
    const TileKernel* pick;    // nullptr: the compute-unit count could not be read
    bool ring_kernel;          // false: the general kernel (K not a multiple of 64, or shorter than three steps)
    int32_t bm, bn, tiles_m, tiles_n_per_tensor, n_cu;
};

// d: features per head; flags: V is flagged for the selection
static LaunchPlan plan_launch(int32_t M, int32_t D, int32_t n_tensors, bool whole_heads, int32_t d, bool flags) {
    static const int n_cu = [] {     // asked once (thread-safe initialisation); 0 = could not be read
        int dev = 0, val = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&val, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        return val;
    }();
    LaunchPlan p{};
    p.n_cu = n_cu;
    if (n_cu <= 0) return p;
    int n_shapes = 0;
    const TileKernel* shapes = tile_shapes(whole_heads, &n_shapes);
    const int forced_tile = (int)tune_value("COCODIFF_GEMM_TILE", 0);     // tuning builds only
    double best = 0.0;
    for (int i = 0; i < n_shapes; ++i) {
        const TileKernel& t = shapes[i];
        if (D / BK < t.min_steps) continue;      // (the rings are filled before the first step)
        if (whole_heads && (d > t.bn || (flags && D > 16 * t.bn))) continue;      // a head spans two wavefronts at most; 16 flag bytes per token tile
        const int64_t tiles = (int64_t)((M + t.bm - 1) / t.bm) * ((D + t.bn - 1) / t.bn) * n_tensors;
        const int64_t rounds = (tiles + n_cu - 1) / n_cu;
        const double cost = (double)rounds * tile_clocks(t, D, whole_heads, (double)tiles / (double)(rounds * n_cu));
        if (forced_tile ? forced_tile == t.bm * 1000 + t.bn : (!p.pick || cost < best)) {
            p.pick = &t;
            best = cost;
        }
    }
    if (!p.pick) p.pick = &shapes[0];
    p.ring_kernel = D % BK == 0 && D >= 3 * BK;
    p.bm = p.ring_kernel ? p.pick->bm : BM;      // the general kernel has one tile shape
    p.bn = p.ring_kernel ? p.pick->bn : BM;
    p.tiles_m = (M + p.bm - 1) / p.bm;
    p.tiles_n_per_tensor = (D + p.bn - 1) / p.bn;
    return p;
}

// Are the chunks, or the fused call's head-parallel V, streamed past the caches, where a later kernel of the step may read them?
//   * A tensor of more than 96 MB has left the last-level cache before it is read, and its dirty lines push the operands out of L2: 20736
//     x 3072, V and then Q and K packed, and their unpack, 951 -> 941 us; the layer in one call at 99840 x 3072 4271 -> 4200, at 40800
//     x 2304 1083 -> 1063.  Of 28 to 57 MB streaming costs that call 0.7 to 1.6 % (the selection reads V from memory).
//   * The chunks of a call for some of the ranks are sent away: one of 12 ranks at 9216 x 3072 71.2 -> 70.3 us, one of 16 at 26112 x
//     2048 69.9 -> 68.0.  (All ranks in one call, so that the unpack reads them: 2144 x 2432 95.3 -> 96.6.)
//   * Chunks are streamed as whole lines or not at all: tiles 192 and 64 features wide have no such kernel (gemm_chunks_streamed.hip).
//   * A fused launch of one round stores everything at its end, and what is dirty then is written back behind it: 1440 x 1216 22.1 ->
//     21.3 us, 3600 x 1152 35.8 -> 35.5, 11248 x 512 36.7 -> 35.8; with a long K loop too, 896 x 3072 58.8 -> 57.5, 1440 x 3072 79.9 ->
//     79.3, of some 2.3 MB 0 to 0.5 % more with everything on chip (384 x 3072, 544 x 2176).  Below 2 MB there is too little of it, and the selection
//     waits for memory (256 x 256 12.0 -> 13.3).
// What counts is what the call writes: its own ranks' rows.  Rotations pair by pair (OUT_FUSED_ANY) have cached stores of V at any size.
static bool streams_outputs(const cocodiff_shape* shape, OutLayout layout, const LaunchPlan& p, bool one_round) {
    const size_t written = (size_t)shape->rank_count * (shape->N / shape->P) * shape->D * 2;
    if (layout == OUT_FUSED) return written > (size_t)96 << 20 || (one_round && written >= (size_t)2 << 20);
    return layout == OUT_CHUNKS && p.pick->entry[OUT_CHUNKS_STREAMED] && (written > (size_t)96 << 20 || shape->rank_count < shape->P);
}

// Workgroups that only fetch operands (fetch_operands), and the column they begin with.
// They take units that a launch of one round leaves idle, 8 of them at least, 32 at most (with 16 launches of 4 to 47 MB are 3 % slower,
// 64 and 128 give the same), from more than 12 K steps on (832 .. 1024 features 2 to 7 % faster, 768 and fewer the same), and where a
// step's loads take as long as its products: tiles of 288 x 192, 224 x 256 and 256 x 256 are -1 to +2 % with them, 192 x 256 -2 to -7 %.
// The tiles read the first column themselves meanwhile (from column 0 on: 4 launches of 12 slower by 10 to 13 %).  Where a column takes
// the fetching units longer than the tiles, they begin further on, so that they are caught up with at the end only (768 x 3072, two
// weights, 16 units: 37.0 us from column 0 on, 33.5 from 1, 31.9 from 2).  Their rate is taken a tenth below kBytesPerClock: fetching
// units that the tiles overtake cost more than they give (432 x 2176, two weights, 18 units: 18.2 us from column 1 on, 15.9 from 2, 17.9
// without any; on chip 14.5, 12.9 and 12.8; fused 256 x 3072, three weights, 32 units: 29.8 from 1, 28.6 from 2, 30.1 without; a
// sixth lower 768 x 3072, two weights, begins from 3: 34.8 alone for 35.4 from 2, but with the rank's other calls 68.5 for 67.7).
// Cold, without and with: 70 launches of one round, 112 .. 9968 tokens x 768 .. 3072 features, one to three weights: 7 % less on average
// (11 % up to 768 tokens), 25 % at most, 1 % more at worst.  (With everything on chip already: fetch_operands.)
// They hold units that another stream's kernel could take meanwhile; what both take together gets shorter all the same (projections of 9
// shapes and permutations side by side, cold, without and with: 768 x 3072, two weights 40.5 and 38.2 us, 1552 x 3072 40.3 and 34.7, 3152 x 1536
// 25.6 and 23.4, 1232 x 1152, three weights 20.1 and 19.6; none longer).
static uint32_t fetching_workgroups(const LaunchPlan& p, int32_t M, int32_t D, int32_t n_tensors, uint32_t n_tiles, uint32_t* from) {
    constexpr uint32_t kAtLeast = 8, kAtMost = 32;
    constexpr int kSteps = 12;
    const uint32_t units = (uint32_t)p.n_cu;
    *from = 0;
    if (!p.ring_kernel || p.pick->per_cu > 1 || D / BK <= kSteps || n_tiles + kAtLeast > units) return 0;
    const double products = tile_mfmas(*p.pick) * 17.2 + 60.0, loads = tile_operand_bytes(*p.pick) / kBytesPerClock;
    if (products > 1.13 * loads) return 0;
    const uint32_t fetchers = std::min(units - n_tiles, kAtMost);
    const double column = ((double)M + (double)n_tensors * D) * kFetchLines * BK * 2.0 / (fetchers * kBytesPerClock / 1.1);
    const int columns = (D / BK + kFetchLines - 1) / kFetchLines;
    *from = (uint32_t)std::max(1, (int)(columns * (1.0 - kFetchLines * std::max(products, loads) / column) + 0.5));
    return fetchers;
}

// How many tile rows tile_at walks together in a fused launch of tiles_m x tiles_n tiles on `workgroups` workgroups.  The operands of
// a launch come from memory when they are read first -- a layer's weights are not on chip -- and a round in which any tile
// reads something new runs at that pace, since a K step's loads are two steps ahead at most.  So the walk is chosen whose first
// round touches every tile row and every column, if there is one: later rounds then find everything in the last-level cache.
// Among those, the one with the fewest operand rows for the XCD that has most.  Else 8 rows: 8 x 4 tiles on an XCD's 32 units,
// close to the least traffic through its L2.
// The whole call, three weights that change from pass to pass, by group size (those that touch everything at once in brackets):
//   2304 x 2560, 15 x 30 tiles   8: 112.1  6: 110.5  5: [105.9]  4: 115.3  3: [106.7] us
//   3072 x 2560, 16 x 30         8: 127.6  6: 126.9  5: [116.1]  4: 126.5  3: [116.8]
//   4608 x 2560, 24 x 30         8: [169.7]  6: 183.9  5: [169.7]  4: [170.8]  3: 184.9
//   4608 x 2816, 29 x 33         8: 234.1  6: [208.3]  5: [206.9]  4: 219.8  3: 209.2
//   2304 x 3072, 12 x 36         8: 136.6  6: 133.9  5: [126.9]  4: [125.3]  3: 136.9
// and with everything on chip 109.5 (8) and 109.6 (4) at 2304 x 3072.
// In one round everything is touched at once.  Where some rows are left over from the groups of 8, the last XCD walks them along all
// columns: 9 rows of 24 columns give it 25 panels of W and the others 3.5, it is the last to end, and fetching workgroups on it
// take from what it waits for.  So a launch with fetching workgroups and more than 8 rows takes the size with the fewest operand rows for
// the XCD that has most, if that is a twentieth less.  The whole call, 8 rows / so, on chip and from memory: 1152 x 2048 38.0 / 35.9 and 42.0 /
// 39.7 us, 544 x 2176 32.5 / 26.0 and 34.7 / 33.5, 1520 x 1024 19.8 / 19.2 and 22.0 / 21.7, 1088 x 2304 42.5 / 41.3 and 45.4 / 45.0; 16 others -3.6 to +0.2 %.  (28 launches without
// fetching workgroups: -3 to +1.5 %, so they stay.)
static uint32_t rows_walked_together(const LaunchPlan& p, uint32_t tiles_n, uint32_t workgroups, bool fetching) {
    const uint32_t tiles_m = (uint32_t)p.tiles_m;
    const uint32_t n_tiles = tiles_m * tiles_n;
    const bool one_round = n_tiles <= workgroups;
    if (tiles_m > 64 || tiles_n > 64 || (one_round && (!fetching || tiles_m <= 8))) return 8;
    const auto bits = [](uint32_t from, uint32_t count) { return (count >= 64 ? ~0ull : (1ull << count) - 1ull) << from; };
    uint32_t best = 8, best_rows = UINT32_MAX;
    for (uint32_t g : {8u, 6u, 5u, 4u, 3u, 7u, 9u, 10u}) {
        if (!one_round && (g == 7 || g > 8)) break;
        uint64_t rows = 0, cols = 0;
        uint32_t most = 0;
        for (uint32_t xcd = 0; xcd < 8; ++xcd) {      // as tiles_of_block deals them out
            const uint32_t per = n_tiles >> 3, rem = n_tiles & 7u;
            uint32_t vt = xcd * per + std::min(xcd, rem);
            const uint32_t end = vt + std::min(per + (xcd < rem ? 1u : 0u), (workgroups >> 3) + (xcd < (workgroups & 7u) ? 1u : 0u));
            uint64_t r = 0, c = 0;
            while (vt < end) {      // group by group, as tile_at walks
                const uint32_t group = vt / (g * tiles_n), first = group * g, high = std::min(tiles_m - first, g);
                const uint32_t from = vt - group * g * tiles_n, to = std::min(end - group * g * tiles_n, high * tiles_n);
                c |= bits(from / high, (to - 1) / high - from / high + 1);
                if (to - from >= high) r |= bits(first, high);
                else
                    for (uint32_t t = from; t < to; ++t) r |= 1ull << (first + t % high);
                vt += to - from;
            }
            rows |= r;
            cols |= c;
            most = std::max(most, (uint32_t)(__builtin_popcountll(r) * p.bm + __builtin_popcountll(c) * p.bn));
        }
        const bool fewer = one_round && g != 8 ? most < best_rows - best_rows / 20 : most < best_rows;
        if (rows == bits(0, tiles_m) && cols == bits(0, tiles_n) && fewer) {
            best = g;
            best_rows = most;
        }
    }
    return best;
}

// What is launched for a call: its tile shape, the workgroups that walk tiles and those that fetch for them, the kernel's layout.
struct Route {
    LaunchPlan plan;
    uint32_t n_tiles, workers, fetchers, fetch_from, group;
    OutLayout layout;
};
static Route route_launch(const cocodiff_shape* shape, int32_t n_tensors, OutLayout layout, bool quad_pairs, bool flags) {
    Route r{};
    const int32_t M = shape->rank_count * (shape->N / shape->P);
    r.plan = plan_launch(M, shape->D, n_tensors, layout == OUT_FUSED, shape->d, flags);
    if (!r.plan.pick) return r;
    r.n_tiles = (uint32_t)r.plan.tiles_m * (uint32_t)r.plan.tiles_n_per_tensor * (uint32_t)n_tensors;
    const uint32_t at_most = (uint32_t)(r.plan.n_cu * r.plan.pick->per_cu);
    r.workers = r.plan.ring_kernel ? std::min(r.n_tiles, at_most) : r.n_tiles;
    r.fetchers = fetching_workgroups(r.plan, M, shape->D, n_tensors, r.n_tiles, &r.fetch_from);
    r.group = layout == OUT_FUSED ? rows_walked_together(r.plan, (uint32_t)r.plan.tiles_n_per_tensor * n_tensors, r.workers, r.fetchers > 0) : 8u;
    r.layout = layout;
    if (layout == OUT_FUSED && !quad_pairs) r.layout = OUT_FUSED_ANY;
    else if (r.plan.ring_kernel && streams_outputs(shape, layout, r.plan, r.n_tiles <= r.workers))
        r.layout = layout == OUT_FUSED ? OUT_FUSED_STREAMED : OUT_CHUNKS_STREAMED;
    return r;
}

}  // namespace cocodiff

using namespace cocodiff;

// layout OUT_SEQ: q, k, v are [N][D]; OUT_CHUNKS: they are exchange buffers, written in chunk order; OUT_HEADS: [H][N][d].
// OUT_FUSED: q, k, v are the exchange buffers and `fused` holds the head-parallel tensors, the gammas and the rotation.
struct FusedExtras {
    cocodiff_bf16* hs[3];              // q_hs, k_hs, v_hs
    const cocodiff_bf16* gamma[2];     // gamma_q, gamma_k
    float eps;
    RopeDev rope;
    // V flagged for the selection on its way out (cocodiff_qkv_proj_fused_select): previous-step V, threshold, flag records
    const cocodiff_bf16* sel_prev;
    uint8_t* sel_flag_bytes;
    float sel_tau;
};

static int proj_launch(const cocodiff_shape* shape, const cocodiff_bf16* x,
                       const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                       cocodiff_bf16* q, cocodiff_bf16* k, cocodiff_bf16* v, OutLayout layout, int slot_order, void* stream,
                       const FusedExtras* fused = nullptr) {
    const bool packed = layout == OUT_CHUNKS || layout == OUT_FUSED;
    int rc = check_shape(shape);
    if (rc != COCODIFF_OK) return rc;
    if (packed && slot_order != COCODIFF_SEND_MAJOR && slot_order != COCODIFF_RECV_MAJOR)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_pack: slot_order (%d) must be SEND_MAJOR or RECV_MAJOR", slot_order);
    if (!x) return fail(COCODIFF_ERR_NULL, "qkv_proj: x is NULL");
    if (fused) {
        const cocodiff_bf16* w3[3] = {wq, wk, wv};
        cocodiff_bf16* b3[3] = {q, k, v};
        for (int i = 0; i < 3; ++i) {
            const bool any_out = b3[i] || fused->hs[i];
            if ((w3[i] != nullptr) != any_out)
                return fail(COCODIFF_ERR_NULL, "qkv_proj_fused: a weight needs at least one of its two outputs, and outputs need their weight");
            if (i < 2 && w3[i] && !fused->gamma[i]) return fail(COCODIFF_ERR_NULL, "qkv_proj_fused: gamma missing for a given Q or K");
            if (!aligned16(fused->hs[i]) || (i < 2 && !aligned16(fused->gamma[i])))
                return fail(COCODIFF_ERR_ALIGN, "qkv_proj_fused: pointers must be 16-byte aligned");
        }
        if (!wq && !wk && !wv) return fail(COCODIFF_ERR_NULL, "qkv_proj_fused: no weight given");
    } else {
        if ((wq == nullptr) != (q == nullptr) || (wk == nullptr) != (k == nullptr) || (wv == nullptr) != (v == nullptr))
            return fail(COCODIFF_ERR_NULL, "qkv_proj: a weight and its output must be given together");
        if (!q && !k && !v) return fail(COCODIFF_ERR_NULL, "qkv_proj: no (weight, output) pair given");
    }
    if (!aligned16(x) || !aligned16(wq) || !aligned16(wk) || !aligned16(wv) || !aligned16(q) || !aligned16(k) || !aligned16(v))
        return fail(COCODIFF_ERR_ALIGN, "qkv_proj: pointers must be 16-byte aligned");

    GemmArgs a;
    a.Ns = (uint32_t)(shape->N / shape->P);
    a.P = (uint32_t)shape->P;
    a.row8 = (uint32_t)(shape->H / shape->P) * (uint32_t)(shape->d / 8);
    a.chunk8 = a.Ns * a.row8;
    a.recv_major = slot_order == COCODIFF_RECV_MAJOR;
    a.N_all = (uint32_t)shape->N;
    a.d8 = (uint32_t)(shape->d / 8);
    a.x = x;
    a.n_tensors = 0;
    const cocodiff_bf16* ws[3] = {wv, wq, wk};   // V first: its tiles are dealt out before Q's and K's
    cocodiff_bf16* ys[3] = {v, q, k};
    cocodiff_bf16* y2s[3] = {fused ? fused->hs[2] : nullptr, fused ? fused->hs[0] : nullptr, fused ? fused->hs[1] : nullptr};
    const cocodiff_bf16* gs[3] = {nullptr, fused ? fused->gamma[0] : nullptr, fused ? fused->gamma[1] : nullptr};
    for (int i = 0; i < 3; ++i) {
        a.w[i] = nullptr;
        a.y[i] = nullptr;
        a.y2[i] = nullptr;
        a.gamma[i] = nullptr;
    }
    for (int i = 0; i < 3; ++i)
        if (ws[i]) {
            a.w[a.n_tensors] = ws[i];
            a.y[a.n_tensors] = ys[i];
            a.y2[a.n_tensors] = y2s[i];
            a.gamma[a.n_tensors] = gs[i];
            ++a.n_tensors;
        }
    a.d = (uint32_t)shape->d;
    a.inv_d = 1.0f / (float)shape->d;
    a.eps = fused ? fused->eps : 0.f;
    a.rope = fused ? fused->rope : RopeDev{};
    a.sel_prev = fused ? fused->sel_prev : nullptr;
    a.sel_flag_bytes = fused ? fused->sel_flag_bytes : nullptr;
    a.sel_th = make_thresholds(fused ? fused->sel_tau : 0.f);
    const int32_t Ns = shape->N / shape->P;
    a.row_begin = shape->rank_begin * Ns;
    a.M = shape->rank_count * Ns;
    a.D = shape->D;
    if (a.D > 1 << 19) return fail(COCODIFF_ERR_SHAPE, "qkv_proj: D (%d) too large", a.D);
    // the four pairs of eight consecutive features are 32 consecutive bytes of a table row when every axis has a multiple of four
    bool quad_pairs = true;
    for (int ax = 0; ax < 3; ++ax) a.row_base[ax] = a.row_stride[ax] = a.row_span[ax] = a.row_end[ax] = a.row_step16[ax] = 0;
    if (layout == OUT_FUSED && (a.gamma[0] || a.gamma[1] || a.gamma[2])) {      // (V alone comes without a rotation)
        uint32_t rest = 16;     // 16 tokens in the grid's mixed radix, last axis fastest
        for (int ax = 2; ax >= 0; --ax) {
            const uint32_t rows = (uint32_t)a.rope.grid[ax];     // absent axes: 0 pairs, 1 row
            if (a.rope.pairs[ax] % 4) quad_pairs = false;
            a.row_base[ax] = (uint32_t)a.rope.offset[ax];
            a.row_stride[ax] = 2u * (uint32_t)a.rope.pairs[ax];
            a.row_span[ax] = rows * a.row_stride[ax];
            a.row_end[ax] = ax < a.rope.n_axes ? a.row_base[ax] + a.row_span[ax] : UINT32_MAX;     // an absent axis never carries
            a.row_step16[ax] = (ax > 0 ? rest % rows : rest) * a.row_stride[ax];
            rest /= rows;
        }
    }
    const Route route = route_launch(shape, a.n_tensors, layout, quad_pairs, a.sel_prev != nullptr);
    const LaunchPlan& plan = route.plan;
    if (!plan.pick) return fail(COCODIFF_ERR_HIP, "qkv_proj: cannot read the compute-unit count");
    if (layout == OUT_FUSED && !plan.ring_kernel)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused: D (%d) must be a multiple of 64 and at least 192", a.D);
    a.bm = plan.bm;
    a.bn = plan.bn;
    a.tiles_m = plan.tiles_m;
    a.tiles_n_per_tensor = plan.tiles_n_per_tensor;
    a.n_tiles = (int32_t)route.n_tiles;
    a.workers = route.workers;
    a.fetch_from = route.fetch_from;
    a.group = route.group;
    // (dividend x divisor below 2^32, as the multiply-high division needs: a weight of more than 2^19 features squared is no
    // memory's)
    a.div_row8 = make_divisor(a.row8);
    a.div_d8 = make_divisor(a.d8);

    // dynamic LDS above 64 KB needs the attribute, once per process (thread-safe initialisation)
    static const hipError_t attr_rc = [] {
        hipError_t e = hipSuccess;
        for (bool whole_heads : {false, true}) {
            int n_shapes = 0;
            const TileKernel* shapes = tile_shapes(whole_heads, &n_shapes);
            for (int i = 0; i < n_shapes; ++i)
                for (const void* k : shapes[i].entry)
                    if (k && e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, shapes[i].lds);
        }
        for (const void* k : {(const void*)qkv_gemm_staged_kernel<OUT_SEQ>, (const void*)qkv_gemm_staged_kernel<OUT_CHUNKS>,
                              (const void*)qkv_gemm_staged_kernel<OUT_HEADS>})
            if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        return e;
    }();
    if (attr_rc != hipSuccess) return fail(COCODIFF_ERR_HIP, "qkv_proj: cannot reserve LDS: %s", hipGetErrorString(attr_rc));
    hipStream_t st = as_stream(stream);
    void* kernel_args[] = {&a};
    hipError_t le;
    static const void* const staged[] = {(const void*)qkv_gemm_staged_kernel<OUT_SEQ>, (const void*)qkv_gemm_staged_kernel<OUT_CHUNKS>,
                                          (const void*)qkv_gemm_staged_kernel<OUT_HEADS>};
    if (plan.ring_kernel)
        le = hipLaunchKernel(plan.pick->entry[route.layout], dim3(route.workers + route.fetchers), dim3(256), kernel_args, plan.pick->lds, st);
    else
        le = hipLaunchKernel(staged[layout], dim3(route.n_tiles), dim3(kStagedThreads), kernel_args, kLdsBytes, st);
    if (le != hipSuccess) return fail(COCODIFF_ERR_HIP, "qkv_proj: launch failed: %s", hipGetErrorString(le));
    return check_launch("qkv_gemm_kernel");
}

extern "C" int cocodiff_qkv_proj(const cocodiff_shape* shape, const cocodiff_bf16* x,
                                 const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                                 cocodiff_bf16* q, cocodiff_bf16* k, cocodiff_bf16* v, void* stream) {
    return proj_launch(shape, x, wq, wk, wv, q, k, v, OUT_SEQ, COCODIFF_SEND_MAJOR, stream);
}

extern "C" int cocodiff_qkv_proj_pack(const cocodiff_shape* shape, const cocodiff_bf16* x,
                                      const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                                      cocodiff_bf16* qbuf, cocodiff_bf16* kbuf, cocodiff_bf16* vbuf, int slot_order, void* stream) {
    return proj_launch(shape, x, wq, wk, wv, qbuf, kbuf, vbuf, OUT_CHUNKS, slot_order, stream);
}

extern "C" int cocodiff_qkv_proj_hs(const cocodiff_shape* shape, const cocodiff_bf16* x,
                                    const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                                    cocodiff_bf16* q_hs, cocodiff_bf16* k_hs, cocodiff_bf16* v_hs, void* stream) {
    return proj_launch(shape, x, wq, wk, wv, q_hs, k_hs, v_hs, OUT_HEADS, COCODIFF_SEND_MAJOR, stream);
}

extern "C" int cocodiff_qkv_proj_fused(const cocodiff_shape* shape, const cocodiff_bf16* x,
                                       const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                                       const cocodiff_bf16* gamma_q, const cocodiff_bf16* gamma_k, float eps, const cocodiff_rope* rope,
                                       cocodiff_bf16* qbuf, cocodiff_bf16* kbuf, cocodiff_bf16* vbuf, int slot_order,
                                       cocodiff_bf16* q_hs, cocodiff_bf16* k_hs, cocodiff_bf16* v_hs, void* stream) {
    int rc = check_shape(shape);
    if (rc != COCODIFF_OK) return rc;
    if (shape->d != 64 && shape->d != 128 && shape->d != 256)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused: d (%d) must be 64, 128 or 256 (a head row must fill whole wavefront tiles of 64 features)", shape->d);
    FusedExtras f{};
    f.hs[0] = q_hs;
    f.hs[1] = k_hs;
    f.hs[2] = v_hs;
    f.gamma[0] = gamma_q;
    f.gamma[1] = gamma_k;
    f.eps = eps;
    if (wq || wk) {
        rc = fill_rope(shape, rope, "qkv_proj_fused", &f.rope);
        if (rc != COCODIFF_OK) return rc;
    }
    return proj_launch(shape, x, wq, wk, wv, qbuf, kbuf, vbuf, OUT_FUSED, slot_order, stream, &f);
}

// Flag records of the projection that flags V: 16 bytes per 16-token tile, one byte per feature tile of V (16 at most; plan_launch
// sees to it with narrower tiles).
static bool flags_in_projection(const cocodiff_shape* shape, int32_t tile_tokens) {
    return tile_tokens == 16 && (shape->D + 255) / 256 <= 16;
}

extern "C" size_t cocodiff_qkv_proj_fused_select_workspace_bytes(const cocodiff_shape* shape, int32_t tile_tokens) {
    if (check_shape(shape) != COCODIFF_OK || tile_tokens <= 0 || shape->N % tile_tokens) return 0;
    if (flags_in_projection(shape, tile_tokens)) return (size_t)(shape->N / 16) * 16;
    return cocodiff_vmajor_select_workspace_bytes(shape->H, shape->N, shape->d, tile_tokens);
}

extern "C" int cocodiff_qkv_proj_fused_select(const cocodiff_shape* shape, const cocodiff_bf16* x,
                                              const cocodiff_bf16* wq, const cocodiff_bf16* wk, const cocodiff_bf16* wv,
                                              const cocodiff_bf16* gamma_q, const cocodiff_bf16* gamma_k, float eps,
                                              const cocodiff_rope* rope,
                                              cocodiff_bf16* qbuf, cocodiff_bf16* kbuf, cocodiff_bf16* vbuf, int slot_order,
                                              cocodiff_bf16* q_hs, cocodiff_bf16* k_hs, cocodiff_bf16* v_hs,
                                              const cocodiff_bf16* v_prev, int32_t tile_tokens, float tau,
                                              int32_t* flags, int32_t* active_idx, int32_t* n_active,
                                              cocodiff_bf16* compact, int32_t cap_tiles,
                                              void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_shape(shape);
    if (rc != COCODIFF_OK) return rc;
    if (shape->rank_begin != 0 || shape->rank_count != shape->P)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused_select: a tile's flag needs every head, so the rank range must be all P ranks");
    if (!wv || !vbuf || !v_hs)
        return fail(COCODIFF_ERR_NULL, "qkv_proj_fused_select: wv, vbuf and v_hs are required (the selection reads V in the head-parallel layout)");
    if (!v_prev || !active_idx || !n_active || !workspace)
        return fail(COCODIFF_ERR_NULL, "qkv_proj_fused_select: v_prev, active_idx, n_active and workspace are required");
    if (!aligned16(v_prev) || !aligned16(workspace) || !aligned16(compact))
        return fail(COCODIFF_ERR_ALIGN, "qkv_proj_fused_select: tensors and workspace must be 16-byte aligned");
    if (tile_tokens <= 0 || shape->N % tile_tokens)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused_select: N (%d) must be a multiple of tile_tokens (%d)", shape->N, tile_tokens);
    if (compact && cap_tiles < 1) return fail(COCODIFF_ERR_CAPACITY, "qkv_proj_fused_select: cap_tiles (%d) must be >= 1", cap_tiles);
    const size_t need = cocodiff_qkv_proj_fused_select_workspace_bytes(shape, tile_tokens);
    if (workspace_bytes < need)
        return fail(COCODIFF_ERR_CAPACITY, "qkv_proj_fused_select: workspace of %zu bytes is smaller than the %zu needed", workspace_bytes, need);
    if (!flags_in_projection(shape, tile_tokens)) {
        // other tile heights, or more than 16 feature tiles: the two calls this one stands for
        rc = cocodiff_qkv_proj_fused(shape, x, wq, wk, wv, gamma_q, gamma_k, eps, rope, qbuf, kbuf, vbuf, slot_order, q_hs, k_hs, v_hs, stream);
        if (rc != COCODIFF_OK) return rc;
        return cocodiff_vmajor_select(shape->H, shape->N, shape->d, tile_tokens, v_hs, v_prev, tau, flags, active_idx, n_active, compact,
                                      cap_tiles, workspace, workspace_bytes, stream);
    }
    if (shape->d != 64 && shape->d != 128 && shape->d != 256)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused: d (%d) must be 64, 128 or 256 (a head row must fill whole wavefront tiles of 64 features)", shape->d);
    FusedExtras f{};
    f.hs[0] = q_hs;
    f.hs[1] = k_hs;
    f.hs[2] = v_hs;
    f.gamma[0] = gamma_q;
    f.gamma[1] = gamma_k;
    f.eps = eps;
    f.sel_prev = v_prev;
    f.sel_flag_bytes = static_cast<uint8_t*>(workspace);
    f.sel_tau = tau;
    if (wq || wk) {
        rc = fill_rope(shape, rope, "qkv_proj_fused_select", &f.rope);
        if (rc != COCODIFF_OK) return rc;
    }
    rc = proj_launch(shape, x, wq, wk, wv, qbuf, kbuf, vbuf, OUT_FUSED, slot_order, stream, &f);
    if (rc != COCODIFF_OK) return rc;
    TileFlags tf;
    tf.words_ptr = static_cast<const uint32_t*>(workspace);
    tf.words = 4;
    const uint32_t bn = (uint32_t)plan_launch(shape->N, shape->D, (wq != nullptr) + (wk != nullptr) + 1, true, shape->d, true).bn;
    const uint32_t parts = ((uint32_t)shape->D + bn - 1u) / bn;        // bytes of a record that the projection wrote
    for (uint32_t w = 0; w < 4; ++w) {
        const uint32_t n = parts > 4 * w ? (parts - 4 * w < 4 ? parts - 4 * w : 4u) : 0u;
        tf.mask[w] = n >= 4 ? 0xffffffffu : (1u << (8 * n)) - 1u;
    }
    return select_finish_launch(shape->H, shape->N, shape->d, tile_tokens, v_hs, tf, flags, active_idx, n_active, compact, cap_tiles, stream);
}

extern "C" int cocodiff_qkv_proj_plan(const cocodiff_shape* shape, int32_t n_tensors, int32_t whole_heads, int32_t* tile_tokens,
                                      int32_t* tile_features, int32_t* n_tiles, int32_t* n_compute_units) {
    int rc = check_shape(shape);
    if (rc != COCODIFF_OK) return rc;
    if (n_tensors < 1 || n_tensors > 3) return fail(COCODIFF_ERR_SHAPE, "qkv_proj_plan: n_tensors (%d) must be 1, 2 or 3", n_tensors);
    const LaunchPlan p = plan_launch(shape->rank_count * (shape->N / shape->P), shape->D, n_tensors, whole_heads != 0, shape->d, false);
    if (!p.pick) return fail(COCODIFF_ERR_HIP, "qkv_proj_plan: cannot read the compute-unit count");
    if (tile_tokens) *tile_tokens = p.bm;
    if (tile_features) *tile_features = p.bn;
    if (n_tiles) *n_tiles = p.tiles_m * p.tiles_n_per_tensor * n_tensors;
    if (n_compute_units) *n_compute_units = p.n_cu;
    return COCODIFF_OK;
}

extern "C" int cocodiff_qkv_proj_route(const cocodiff_shape* shape, int32_t n_tensors, int32_t form, int32_t* tile_tokens, int32_t* tile_features,
                                       int32_t* n_tiles, int32_t* fetching, int32_t* fetch_from, int32_t* streamed, int32_t* rows_together) {
    int rc = check_shape(shape);
    if (rc != COCODIFF_OK) return rc;
    if (n_tensors < 1 || n_tensors > 3) return fail(COCODIFF_ERR_SHAPE, "qkv_proj_route: n_tensors (%d) must be 1, 2 or 3", n_tensors);
    if (form < 0 || form > 4) return fail(COCODIFF_ERR_SHAPE, "qkv_proj_route: form (%d) must be 0 .. 4", form);
    const OutLayout layout = form == 0 ? OUT_SEQ : form == 1 ? OUT_CHUNKS : form == 2 ? OUT_HEADS : OUT_FUSED;
    const Route r = route_launch(shape, n_tensors, layout, true, form == 4 && flags_in_projection(shape, 16));
    if (!r.plan.pick) return fail(COCODIFF_ERR_HIP, "qkv_proj_route: cannot read the compute-unit count");
    if (layout == OUT_FUSED && (!r.plan.ring_kernel || (shape->d != 64 && shape->d != 128 && shape->d != 256)))
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_route: no fused projection of D (%d) in heads of %d", shape->D, shape->d);
    if (tile_tokens) *tile_tokens = r.plan.bm;
    if (tile_features) *tile_features = r.plan.bn;
    if (n_tiles) *n_tiles = (int32_t)r.n_tiles;
    if (fetching) *fetching = (int32_t)r.fetchers;
    if (fetch_from) *fetch_from = (int32_t)r.fetch_from;
    if (streamed) *streamed = r.layout == OUT_CHUNKS_STREAMED || r.layout == OUT_FUSED_STREAMED;
    if (rows_together) *rows_together = (int32_t)r.group;
    return COCODIFF_OK;
}
