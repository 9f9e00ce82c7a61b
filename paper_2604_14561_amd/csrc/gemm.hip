// QKV projection (paper Section II-B): Y[n][o] = sum_k X[n][k] * W[o][k], bf16 in, fp32 accumulate on the
// gfx950 matrix cores, one RNE rounding to bf16.  The main kernel multiplies with v_mfma_f32_16x16x32_bf16: on this
// power-limited part it sustains 1.91 PFLOP/s at 0.70 pJ/flop in a register-only loop against 1.72 PFLOP/s at
// 0.77 pJ/flop for v_mfma_f32_32x32x16_bf16, for the same LDS traffic per flop (a wavefront's tile decides that).
//
// Workgroup tile (tokens x features): 256 x 256, 288 x 192 or 192 x 192 -- the host takes the one with the fewest
// rounds of tiles over the compute units, weighted by a measured per-flop cost (plan_launch).  K step 64: a row
// segment of either operand is one whole 128-byte line (half lines halve the L1 fill rate).  W rides the MFMA "A"
// side, so an accumulator lane holds four consecutive features of one token.  Both operands are K-contiguous; LDS
// tiles keep rows contiguous and store 16-byte column c of row r at column c ^ swz(r), which makes the 128-bit
// fragment reads bank-conflict free.
//
// Main kernel (K a multiple of 64, at least three steps): global -> LDS directly (no staging registers) through two
// rings, three slots for X tiles and two for W tiles (160 KB for the 256 x 256 tile).  Eight wavefronts, four along
// the features x two along the tokens, two per SIMD, so one can multiply while the other waits for LDS, memory or
// the barrier.  General kernel (any K that is a multiple of 8): global -> registers -> LDS, zero-filled K tail.
// The epilogue rounds to bf16, transposes through the (now idle) LDS and writes 16-byte vectors: rows of [N][D],
// row pieces straight into their chunks of the exchange buffer, or row pieces of the head-parallel tensor -- or, in
// the fused form (tiles 256 features wide, so that they hold whole heads), it first RMS-normalises and rotates Q and K
// on the fp32 accumulators (paper Section II-B's norm and RoPE, one rounding in all) and writes both the chunks and
// the head-parallel tensor.
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace cocodiff {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int BM = 256;          // tokens per workgroup tile
constexpr int BK = 64;           // K elements per step
constexpr int kTileBytes = BM * BK * 2;                  // one operand tile of one K step of the fallback kernel: 32 KB
constexpr int kStageBytes = 2 * kTileBytes;              // 64 KB
constexpr int kLdsBytes = 2 * kStageBytes;               // 128 KB

struct GemmArgs {
    const uint16_t* x;
    const uint16_t* w[3];
    uint16_t* y[3];
    int32_t n_tensors;
    int32_t row_begin, M;      // token rows [row_begin, row_begin + M)
    int32_t D;                 // features per tensor = K
    int32_t tiles_m, tiles_n_per_tensor, n_tiles;
    int32_t bm, bn;            // tile of the launch: tokens x features
    // outputs in exchange-buffer (chunk) order instead of [N][D]: tokens per rank, ranks, 16-byte vectors per
    // chunk row and per chunk, slot order
    uint32_t Ns, P, row8, chunk8;
    int32_t recv_major;
    // outputs in head-parallel order [H][N][d]: all tokens, 16-byte vectors per head row
    uint32_t N_all, d8;
    // OUT_FUSED: second destination (head-parallel; y[] is then the exchange buffer; either may be null), RMSNorm + RoPE
    // of the tensors that have a gamma
    uint16_t* y2[3];
    const uint16_t* gamma[3];
    uint32_t d;                // features per head
    float inv_d, eps;
    RopeDev rope;
    // How the normalising epilogue walks the rotation table, in floats: axis x' rows start at row_base[x], row_stride[x]
    // apart, row_span[x] = grid x stride in all, up to row_end[x] (absent axes: never reached); row_step16[x] = the axis'
    // digit of 16 tokens in the grid's mixed radix (last axis fastest) times the stride.
    uint32_t row_base[3], row_stride[3], row_span[3], row_end[3], row_step16[3];
    Divisor div_row8, div_d8;  // by row8 and by d8 (dividends below D/8)
    // The fused call that also flags V for the selection (sel_prev != nullptr): the previous step's V in the head-parallel
    // layout, the decision's thresholds, and the flag records: 16 bytes per 16-token tile, byte c written by the workgroup
    // of V's feature tile c.
    const uint16_t* sel_prev;
    uint8_t* sel_flag_bytes;
    Thresholds sel_th;
};

// Where the epilogue writes: token-major [N][D]; the exchange-buffer chunks of the first all-to-all; or the
// head-parallel tensor [H][N][d] that all-to-all ends in (pack, exchange and unpack folded into the store address).
// OUT_FUSED: Q and K are normalised and rotated in the epilogue (on the fp32 accumulators), and every tensor goes to its
// exchange buffer and to its head-parallel tensor (whichever are given).
// OUT_FUSED_ANY: the same for rotations in which an axis' pairs are not a multiple of four (pair by pair through the table).
enum OutLayout { OUT_SEQ = 0, OUT_CHUNKS = 1, OUT_HEADS = 2, OUT_FUSED = 3, OUT_FUSED_ANY = 4 };

// [rows][64] bf16 tiles (128-byte rows): any 16 consecutive rows of one column land in 16 different
// 16-byte slots of the 256-byte bank span.
__device__ __forceinline__ uint32_t swz(uint32_t row) { return (row & 7u) ^ ((row >> 3) & 1u); }

// Byte offset of 16-byte column c of row r inside a [rows][64] bf16 LDS tile.
__device__ __forceinline__ uint32_t lds_off(uint32_t row, uint32_t c) { return row * 128u + ((c ^ swz(row)) << 4); }

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

struct TileCoord {
    uint32_t tensor, m0, f0;
};

// Tile `vt` of the launch: groups of 8 tile rows walked column by column, so that tiles with neighbouring numbers share rows
// of X and W.
__device__ __forceinline__ TileCoord tile_at(const GemmArgs& a, uint32_t vt) {
    const uint32_t tiles_n = (uint32_t)a.tiles_n_per_tensor * a.n_tensors;
    constexpr uint32_t GROUP = 8;
    const uint32_t per_group = GROUP * tiles_n;
    const uint32_t grp = vt / per_group;
    const uint32_t first_m = grp * GROUP;
    const uint32_t rows_here = min((uint32_t)a.tiles_m - first_m, GROUP);
    const uint32_t in_grp = vt - grp * per_group;
    const uint32_t tm = first_m + in_grp % rows_here;
    const uint32_t tn = in_grp / rows_here;
    TileCoord t;
    t.tensor = tn / a.tiles_n_per_tensor;
    t.m0 = tm * (uint32_t)a.bm;
    t.f0 = (tn - t.tensor * a.tiles_n_per_tensor) * (uint32_t)a.bn;
    return t;
}

// Blocks are dealt round-robin to the 8 XCDs: XCD x takes a contiguous run of the tiles, so that tiles running together share
// rows of X and W in that XCD's L2.  A workgroup takes tile `first`, then every `stride`-th one below `end`.
struct TileWalk {
    uint32_t first, end, stride;
};
__device__ __forceinline__ TileWalk tiles_of_block(const GemmArgs& a) {
    const uint32_t n_tiles = (uint32_t)a.n_tiles, xcd = blockIdx.x & 7u;
    const uint32_t per = n_tiles >> 3, rem = n_tiles & 7u;   // XCD x gets per + (x < rem) tiles
    const uint32_t begin = xcd * per + min(xcd, rem);
    return {begin + (blockIdx.x >> 3), begin + per + (xcd < rem ? 1u : 0u), (gridDim.x >> 3) + (xcd < (gridDim.x & 7u) ? 1u : 0u)};
}

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

// The accumulators live in the accumulation registers a0 .. a255 by number, and the compiler does not know them: accumulator
// tile (i, j) is a[4 (i NJ + j)] and the three behind it.  (Left to the compiler, it moves accumulators between the two
// register files and to scratch memory -- at 256 of them the loops over K steps and tiles carry 128 moves each way per step.)
// What the compiler may not do is keep something of its own there: reserve_accumulators() in every K step and every token
// tile of the epilogue tells it that all of them change.  The waits that these instructions need are in the code too: an MFMA
// result is read only behind mfma_results_ready(), and many instructions lie between clearing an accumulator and the next MFMA
// on it.
#define COCODIFF_ALL_ACC \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", \
    "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", \
    "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", \
    "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", \
    "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", \
    "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", \
    "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", \
    "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", \
    "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", \
    "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", \
    "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", \
    "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", \
    "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", \
    "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211", "a212", "a213", \
    "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225", "a226", "a227", \
    "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", "a240", "a241", \
    "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
__device__ __forceinline__ void reserve_accumulators() { asm volatile("" ::: COCODIFF_ALL_ACC); }
template <int AT>
__device__ __forceinline__ void mfma_acc(const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(w), "v"(x), "n"(AT), "n"(AT + 3));
}
template <int AT>
__device__ __forceinline__ float read_acc() {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(AT));
    return x;
}
// Between a vector instruction that writes a register and an MFMA that reads it lie two wait states at least.
__device__ __forceinline__ void mfma_operands_ready() {
    asm volatile("s_nop 1" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ bf16x8 zero_fragment() {
    bf16x8 z = __builtin_bit_cast(bf16x8, vec16{0u, 0u, 0u, 0u});
    asm volatile("s_nop 1" : "+v"(z));      // (opaque: not written anew in front of every use)
    return z;
}
// Accumulator tile AT .. AT + 3 to zero: a product of zeros on the matrix core (one instruction where four register writes
// would do the same).
template <int AT>
__device__ __forceinline__ void clear_acc(const bf16x8& zero) {
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], %0, %0, 0" ::"v"(zero), "n"(AT), "n"(AT + 3));
}
// eight wait states of the 16-pass MFMA and more
__device__ __forceinline__ void mfma_results_ready() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
// f(std::integral_constant<int, 0>{}), ..., f(N - 1): a loop whose index is a template argument
template <int... I, typename F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) { for_each_index(std::make_integer_sequence<int, N>{}, f); }

// ---- epilogue of the main kernel ------------------------------------------------------------------------------------
// W's rows are loaded into LDS in an order (w_row_of) that leaves a lane, in the accumulator tiles 2p and 2p + 1 of a token
// tile, with EIGHT consecutive features of one token: lane l has features 32 p + 8 (l / 16) .. + 7 of the wavefront's, token
// l % 16 of the token tile -- one 16-byte vector, so nothing goes through LDS on the way out and the ring is free to take
// the next tile's operands meanwhile.  A store instruction writes 64 consecutive bytes of sixteen tokens.
// Sizes are kind: token ranges start and end at multiples of 16 and the launch's D is a multiple of 64, so a token tile or a
// group of 32 features exists as a whole or not at all, and a token tile lies in one rank's chunk.  A destination address is
// therefore a per-lane part (feature, token within the token tile: formed once) plus a part that is the same for the
// wavefront (token tile), stepped by scalar instructions.
__device__ __forceinline__ uint32_t w_row_of(uint32_t lds_row) {
    return (lds_row & ~31u) + ((lds_row & 12u) << 1) + ((lds_row & 16u) >> 2) + (lds_row & 3u);
}

// Where a wavefront's vectors go, in 16-byte vectors from the tensor's start: lane part by group of 32 features, then the
// token tile's part.
template <int NP>
struct Dest {
    size_t lane[NP];
};

// [N][D]
template <int NP>
__device__ __forceinline__ Dest<NP> dest_seq(const GemmArgs& a, uint32_t v8, uint32_t tl) {
    Dest<NP> t;
#pragma unroll
    for (int p = 0; p < NP; ++p) t.lane[p] = (size_t)tl * ((uint32_t)a.D / 8u) + v8 + 4u * p;
    return t;
}
// exchange buffer: vector v of token n = r*Ns + m belongs to chunk (sender r, receiver v / row8), row m, column v % row8
template <int NP>
__device__ __forceinline__ Dest<NP> dest_chunks(const GemmArgs& a, uint32_t v8, uint32_t tl) {
    Dest<NP> t;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t v = v8 + 4u * p, rcv = div_by<true>(v, a.div_row8), c = v - rcv * a.row8;
        t.lane[p] = (size_t)(a.recv_major ? rcv * a.P : rcv) * a.chunk8 + tl * a.row8 + c;
    }
    return t;
}
// [H][N][d]
template <int NP>
__device__ __forceinline__ Dest<NP> dest_heads(const GemmArgs& a, uint32_t v8, uint32_t tl) {
    Dest<NP> t;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t v = v8 + 4u * p, h = div_by<true>(v, a.div_d8), c = v - h * a.d8;
        t.lane[p] = (size_t)h * a.N_all * a.d8 + tl * a.d8 + c;
    }
    return t;
}

// The token tile's part of an exchange-buffer address, stepped from one token tile to the next.
struct ChunkWalk {
    uint32_t m;
    size_t at;
    __device__ __forceinline__ ChunkWalk(const GemmArgs& a, uint32_t n) {
        const uint32_t r = n / a.Ns;
        m = n - r * a.Ns;
        at = (size_t)(a.recv_major ? r : r * a.P) * a.chunk8 + (size_t)m * a.row8;
    }
    __device__ __forceinline__ void next(const GemmArgs& a) {      // 16 tokens on, into the next sender's chunk where m reaches Ns
        m += 16u;
        at += (size_t)16u * a.row8;
        if (m >= a.Ns) {
            m = 0;
            at += a.recv_major ? 0 : (size_t)(a.P - 1u) * a.chunk8;
        }
    }
};

__device__ __forceinline__ vec16 pack_vec(const float (&x)[8]) {
    return vec16{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
}

// A wavefront's part of a tile on its way out: how many token tiles and groups of 32 features exist, global index of its first
// token, the lane's token within a token tile, the lane's vector of feature group 0 within a token row of the tensor.
struct TileOut {
    int live_j, live_p;
    uint32_t n0, tl, v8;
};

// The lane's vector of feature group P and token tile J.
template <int NJ, int P, int J>
__device__ __forceinline__ void take_acc(float (&x)[8]) {
    unrolled<8>([&](auto e_c) __attribute__((always_inline)) {
        constexpr int e = decltype(e_c)::value;
        x[e] = read_acc<4 * ((2 * P + e / 4) * NJ + J) + e % 4>();
    });
}
// f(token tile, a constant) for those that exist; the accumulators are cleared for the workgroup's next tile.
template <int NI, int NJ, typename F>
__device__ __forceinline__ void for_token_tiles(const TileOut& t, F&& f) {
    const bf16x8 zero = zero_fragment();
    unrolled<NJ>([&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        reserve_accumulators();
        if (j < t.live_j && t.live_p > 0) f(j_c);
        unrolled<NI>([&](auto i_c) __attribute__((always_inline)) { clear_acc<4 * (decltype(i_c)::value * NJ + j)>(zero); });
    });
}
// The vectors of one token tile to y (features come in groups of 64: the two halves of a wavefront's exist or do not).
template <bool NT, int NP>
__device__ __forceinline__ void store_groups(vec16* __restrict__ y, const Dest<NP>& to, const vec16 (&v)[NP], int live_p) {
    if (live_p == NP) {
#pragma unroll
        for (int p = 0; p < NP; ++p) st_vec<NT>(y + to.lane[p], v[p]);
    } else {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (p < live_p) st_vec<NT>(y + to.lane[p], v[p]);
    }
}

// Sum over the four lanes that hold one token's features (lanes l, l+16, l+32, l+48), in all four.
__device__ __forceinline__ float sum_of_token(float s) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Stores.  Cache policy: what a kernel of the same step reads next stays cached -- [N][D], the head-parallel V (the
// selection reads it), and the exchange buffer of cocodiff_qkv_proj_pack (its unpack follows).  In the fused call nothing on
// this GPU reads the exchange buffers (they are what the all-to-all would send) or, within the step, the head-parallel Q and
// K: streamed past the caches they leave nothing dirty in L2 to be written back under the next round's loads.
template <int NI, int NJ, int LAYOUT>
__device__ __forceinline__ void store_plain(const GemmArgs& a, const TileOut& t, uint16_t* __restrict__ Y) {
    constexpr int NP = NI / 2;
    const Dest<NP> to = LAYOUT == OUT_SEQ ? dest_seq<NP>(a, t.v8, t.tl) : LAYOUT == OUT_CHUNKS ? dest_chunks<NP>(a, t.v8, t.tl) : dest_heads<NP>(a, t.v8, t.tl);
    ChunkWalk chunk(a, t.n0);
    const uint32_t row = LAYOUT == OUT_SEQ ? (uint32_t)a.D / 8u : a.d8;
    vec16* y = reinterpret_cast<vec16*>(Y) + (LAYOUT == OUT_CHUNKS ? 0 : (size_t)t.n0 * row);
    for_token_tiles<NI, NJ>(t, [&](auto j_c) __attribute__((always_inline)) {
        vec16 v[NP];
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            float x[8];
            take_acc<NJ, decltype(p_c)::value, decltype(j_c)::value>(x);
            v[decltype(p_c)::value] = pack_vec(x);
        });
        if (LAYOUT == OUT_CHUNKS) {
            store_groups<false>(y + chunk.at, to, v, t.live_p);
            chunk.next(a);
        } else {
            store_groups<false>(y, to, v, t.live_p);
            y += (size_t)16u * row;
        }
    });
}

// Both destinations of the fused call (V): Y the exchange buffer, Y2 the head-parallel tensor (either may be null).
// SELECT: the selection's flags are wanted too (paper Section III-D; both destinations are given): every vector on its way out
// is compared with the previous step's vector at the same place of the head-parallel layout.  The fp32 difference decides
// unless its magnitude is exactly the threshold's (internal.h), so a lane needs only the largest magnitude of a token tile,
// taken on the bit patterns (a NaN is then larger than any number); a token tile whose largest magnitude ties with the
// threshold -- practically never -- is compared again in double, from memory, when everything is stored.  The previous
// vectors of a token tile are fetched AHEAD token tiles before it.  Returns, the same in every lane, a bit per token tile: did
// any of the wavefront's vectors change?
template <int NI, int NJ, bool SELECT>
__device__ __forceinline__ uint32_t store_both(const GemmArgs& a, const TileOut& t, uint16_t* __restrict__ Y, uint16_t* __restrict__ Y2) {
    constexpr int NP = NI / 2, AHEAD = 2;
    const Dest<NP> to_c = dest_chunks<NP>(a, t.v8, t.tl), to_h = dest_heads<NP>(a, t.v8, t.tl);
    ChunkWalk chunk(a, t.n0);
    const size_t at0 = (size_t)t.n0 * a.d8, step = (size_t)16u * a.d8;
    vec16 *yc = reinterpret_cast<vec16*>(Y), *yh = reinterpret_cast<vec16*>(Y2) + at0;
    const vec16* yp = reinterpret_cast<const vec16*>(a.sel_prev) + at0;
    vec16 prev[AHEAD + 1][NP];
    auto fetch = [&](int j) __attribute__((always_inline)) {
        if (SELECT && j < t.live_j) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (p < t.live_p) prev[j % (AHEAD + 1)][p] = ld_nt(yp + step * j + to_h.lane[p]);
        }
    };
#pragma unroll
    for (int j = 0; j < AHEAD && j < NJ; ++j) fetch(j);
    uint32_t verdict = 0, ties = 0;
    for_token_tiles<NI, NJ>(t, [&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        if constexpr (j + AHEAD < NJ) fetch(j + AHEAD);
        vec16 v[NP];
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            float x[8];
            take_acc<NJ, decltype(p_c)::value, j>(x);
            v[decltype(p_c)::value] = pack_vec(x);
        });
        if (Y) store_groups<true>(yc + chunk.at, to_c, v, t.live_p);
        if (Y2) store_groups<false>(yh, to_h, v, t.live_p);
        if (SELECT) {
            uint32_t largest = 0;
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (p < t.live_p) largest = max(largest, vec_largest_difference(v[p], prev[j % (AHEAD + 1)][p]));
            verdict |= (__ballot(a.sel_th.always || largest > a.sel_th.tau_bits) != 0 ? 1u : 0u) << j;
            ties |= (__ballot(largest == a.sel_th.tie_bits) != 0 ? 1u : 0u) << j;
        }
        chunk.next(a);
        yh += step;
    });
    if (SELECT) {
        ties &= ~verdict;
        while (ties) {
            const int j = __builtin_ctz(ties);
            ties &= ties - 1u;
            const vec16* now = reinterpret_cast<const vec16*>(Y2) + at0 + step * j;
            bool changed = false;
            for (int p = 0; p < t.live_p; ++p) {
                const uint32_t v = t.v8 + 4u * p, h = v / a.d8;
                const size_t at = (size_t)h * a.N_all * a.d8 + t.tl * a.d8 + (v - h * a.d8);
                changed |= vec_changed_double(now[at], yp[step * j + at], a.sel_th.tau);
            }
            verdict |= (__ballot(changed) != 0 ? 1u : 0u) << j;
        }
    }
    return verdict;
}

// RMSNorm over every head row and RoPE on the fp32 accumulators, in the arithmetic order of the stand-alone norm + RoPE
// kernel (x * rinv * gamma, then the rotation) -- but on the unrounded projection, so Q and K are rounded to bf16 once
// instead of twice -- and out to both destinations.
// A wavefront holds 128 features of its tokens: two heads of 64, one of 128, or half of one of 256, whose sums of squares
// the two wavefronts exchange through `xch` (LDS, [wavefront][token]; two workgroup barriers, the second so that nobody
// overwrites what the other still reads).
// This stage's time is its instruction count (nothing else runs on the unit meanwhile), so the token's grid coordinates are
// divided out once, for token tile 0, and then stepped as table row offsets: 16 tokens further is a.row_step16[] further in
// mixed radix, with carries (the absent axes of a one- or two-axis grid are grids of one cell: they never carry).  The
// (cos, sin) values of a token tile are fetched from the table (L1 / L2) while its sums of squares are formed.
// QUADS: every axis has a multiple of four pairs, so the four pairs of a vector are 32 consecutive bytes of a table row.
template <int NI, int NJ, bool QUADS>
__device__ __forceinline__ void store_normalised(const GemmArgs& a, const TileOut& t, const uint16_t* __restrict__ gamma, uint16_t* __restrict__ Y,
                                                 uint16_t* __restrict__ Y2, float* xch, uint32_t wave) {
    constexpr int NP = NI / 2;
    constexpr uint32_t WF = NI * 16;                 // features per wavefront
    static_assert(NP == 4, "the wavefront's features are two halves of 64");
    const bool wide = a.d > WF;                      // a head of two wavefronts; the same for the whole launch
    if (wide) {
        unrolled<NJ>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value;
            reserve_accumulators();
            float s = 0.f;
            unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
                float x[8];
                take_acc<NJ, decltype(p_c)::value, j>(x);
#pragma unroll
                for (int e = 0; e < 8; ++e) s += x[e] * x[e];
            });
            s = sum_of_token(s);
            xch[wave * (NJ * 16) + 16 * j + t.tl] = s;      // (four lanes, one value)
        });
        __syncthreads();
    }

    // the lane's four rotary pairs of feature group p: which axis' table, and the float offset inside a table row
    const uint32_t p0 = (uint32_t)a.rope.pairs[0], p01 = p0 + (uint32_t)a.rope.pairs[1];
    auto axis_of = [&](uint32_t pr) __attribute__((always_inline)) { return a.rope.n_axes > 2 && pr >= p01 ? 2u : a.rope.n_axes > 1 && pr >= p0 ? 1u : 0u; };
    uint32_t pair0[NP];                              // index inside the head of the group's first pair
    vec16 g[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t fh = (8u * (t.v8 + 4u * p)) & (a.d - 1u);      // d is 64, 128 or 256
        pair0[p] = fh / 2u;
        g[p] = *reinterpret_cast<const vec16*>(gamma + fh);
    }
    // float offsets of the token's row in each axis' table, for this lane's token of token tile 0 (axes 1 and 2: less the pairs
    // before them)
    uint32_t row_a[3];
    {
        uint32_t rem = t.n0 + t.tl;
        const uint32_t c2 = rem % (uint32_t)a.rope.grid[2];
        rem /= (uint32_t)a.rope.grid[2];
        const uint32_t c1 = rem % (uint32_t)a.rope.grid[1];
        rem /= (uint32_t)a.rope.grid[1];
        row_a[0] = a.row_base[0] + rem * a.row_stride[0];
        row_a[1] = a.row_base[1] + c1 * a.row_stride[1];
        row_a[2] = a.row_base[2] + c2 * a.row_stride[2];
    }
    const float* cs_table = a.rope.cs;
    auto load_cs = [&](float (&to)[NP][8]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (QUADS) {
                const uint32_t ax = axis_of(pair0[p]);
                const uint32_t off = (ax == 0 ? row_a[0] : ax == 1 ? row_a[1] - 2u * p0 : row_a[2] - 2u * p01) + 2u * pair0[p];
                const float4 lo = *reinterpret_cast<const float4*>(cs_table + off), hi = *reinterpret_cast<const float4*>(cs_table + off + 4u);
                to[p][0] = lo.x; to[p][1] = lo.y; to[p][2] = lo.z; to[p][3] = lo.w;
                to[p][4] = hi.x; to[p][5] = hi.y; to[p][6] = hi.z; to[p][7] = hi.w;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t pr = pair0[p] + q, ax = axis_of(pr);
                    const uint32_t off = (ax == 0 ? row_a[0] : ax == 1 ? row_a[1] - 2u * p0 : row_a[2] - 2u * p01) + 2u * pr;
                    const float2 c = *reinterpret_cast<const float2*>(cs_table + off);
                    to[p][2 * q] = c.x;
                    to[p][2 * q + 1] = c.y;
                }
            }
        }
    };
    auto next_token_tile = [&]() __attribute__((always_inline)) {
        row_a[2] += a.row_step16[2];
        const bool carry2 = row_a[2] >= a.row_end[2];
        row_a[2] -= carry2 ? a.row_span[2] : 0u;
        row_a[1] += a.row_step16[1] + (carry2 ? a.row_stride[1] : 0u);
        const bool carry1 = row_a[1] >= a.row_end[1];
        row_a[1] -= carry1 ? a.row_span[1] : 0u;
        row_a[0] += a.row_step16[0] + (carry1 ? a.row_stride[0] : 0u);
    };

    const Dest<NP> to_c = dest_chunks<NP>(a, t.v8, t.tl), to_h = dest_heads<NP>(a, t.v8, t.tl);
    ChunkWalk chunk(a, t.n0);
    vec16 *yc = reinterpret_cast<vec16*>(Y), *yh = reinterpret_cast<vec16*>(Y2) + (size_t)t.n0 * a.d8;
    const bool two_heads = a.d < WF;
    for_token_tiles<NI, NJ>(t, [&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        float cs[NP][8];
        load_cs(cs);
        next_token_tile();
        float x[NP][8], s[2] = {0.f, 0.f};
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            take_acc<NJ, p, j>(x[p]);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[p / 2] += x[p][e] * x[p][e];
        });
        float rinv[2];
        if (two_heads) {
#pragma unroll
            for (int u = 0; u < 2; ++u) rinv[u] = 1.0f / sqrtf(sum_of_token(s[u]) * a.inv_d + a.eps);
        } else {
            const float ss = wide ? xch[(wave & ~1u) * (NJ * 16) + 16 * j + t.tl] + xch[(wave | 1u) * (NJ * 16) + 16 * j + t.tl]
                                  : sum_of_token(s[0] + s[1]);
            rinv[0] = rinv[1] = 1.0f / sqrtf(ss * a.inv_d + a.eps);
        }
        vec16 v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t gw[4] = {g[p].x, g[p].y, g[p].z, g[p].w};
            float o[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float ev = x[p][2 * q] * rinv[p / 2] * bf16_lo(gw[q]);
                const float od = x[p][2 * q + 1] * rinv[p / 2] * bf16_hi(gw[q]);
                o[2 * q] = ev * cs[p][2 * q] - od * cs[p][2 * q + 1];
                o[2 * q + 1] = ev * cs[p][2 * q + 1] + od * cs[p][2 * q];
            }
            v[p] = pack_vec(o);
        }
        if (Y) store_groups<true>(yc + chunk.at, to_c, v, t.live_p);
        if (Y2) store_groups<true>(yh, to_h, v, t.live_p);
        chunk.next(a);
        yh += (size_t)16u * a.d8;
    });
    if (wide) __syncthreads();      // before anybody loads into the exchange's slot again
}

// s_waitcnt: at most WAIT global->LDS loads of this wavefront still in flight (LDS-read counter untouched)
template <int WAIT>
__device__ __forceinline__ void wait_loads() {
    static_assert(WAIT >= 0 && WAIT < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (WAIT & 15) | ((WAIT >> 4) << 14));
}
// the same, and every LDS read has returned
template <int WAIT>
__device__ __forceinline__ void wait_loads_and_lds() {
    __builtin_amdgcn_s_waitcnt(0x0070 | (WAIT & 15) | ((WAIT >> 4) << 14));
}

// ---------------------------------------------------------------------------------------------
// Main kernel.  A step's X tile and W tile travel through two rings in LDS: three slots for X (X of K step kt in
// slot kt % 3) and two for W (slot kt % 2) -- 160 KB for a 256 x 256 tile (five times 32 KB), 156 KB for 288 tokens x
// 192 features (3 x 36 + 2 x 24 KB).  A K step is two halves of 32 K elements, one v_mfma_f32_16x16x32_bf16 per
// 16 x 16 output tile and half.  In step kt a wavefront multiplies half 0 while reading the fragments of half 1,
// waits until step kt+1 has landed (its own loads; the barrier covers the other wavefronts'), then multiplies half 1
// while reading half 0 of step kt+1.  After that barrier every wavefront is past its last read of step kt, so W of
// step kt+2 goes into the W slot of step kt (during half 1 of step kt) and X of step kt+3 into its X slot (during
// half 0 of step kt+1).  The loads are issued one at a time between the MFMAs: a wavefront that issues its eight
// loads of a step in one burst stalls on the address unit, and the MFMAs behind them in program order with it
// (measured: +340 cycles per step).
// The MFMAs of a half run token tile by token tile: the X fragment of a token tile is dead after NI MFMAs and is
// read again for the next half right there (X fragments need one register set), the NI W fragments live through
// the half and have two sets.  Instruction order inside a half is pinned by a scheduling barrier after every
// instruction group.
// ---------------------------------------------------------------------------------------------
constexpr int kXSlots = 3, kWSlots = 2;
constexpr double kPenalty288 = 1.07;   // measured per-flop cost of the 288 x 192 tile against 256 x 256 (4.5 - 8 %):
                                       // 11 % more operand bytes into LDS and 18 % more fragment reads per flop
constexpr double kPenalty192 = 1.2;    // 192 x 192: a third more operand bytes and twice the fragment reads per flop
constexpr int ring_lds_bytes(int bm, int bn) { return (kXSlots * bm + kWSlots * bn) * BK * 2; }
// One global -> LDS load of 16 bytes per lane: lane l's vector lands at lds_addr + 16*l.  Written as inline
// assembly so that the compiler does not tie later LDS reads to it with a full vmcnt wait (it cannot tell
// that the ring slot being filled is not the one being read); completion is awaited by wait_loads().
// Two instructions, so that the wavefront can multiply in between: M0 takes the LDS address, then the load is issued (nothing
// else in the kernel uses M0; an instruction has to lie between the two).
template <int PLUS>
__device__ __forceinline__ void load_dest(uint32_t lds_addr) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(lds_addr), "n"(PLUS) : "memory", "m0", "scc");
}
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off) {
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base) : "memory");
}

// The kernel's arguments, read again from where the launch put them: what only the epilogue needs does not stay in scalar
// registers (of which there are too few) through the K loop.
__device__ __forceinline__ const GemmArgs& arguments_again() {
    uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const GemmArgs*)(const __attribute__((address_space(4))) GemmArgs*)at;
}

// Scalar steps of the K loop, kept where they are written.
__device__ __forceinline__ void set_scalar(uint32_t& to, uint32_t from) { asm volatile("s_mov_b32 %0, %1" : "=s"(to) : "s"(from)); }

// The workgroup's barrier without the fence of __syncthreads() (which drains the LDS reads in flight): what has to have
// completed is waited for in front of it.
__device__ __forceinline__ void wave_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Tile = (2 * NJ * 16) tokens x (WN * NI * 16) features, WN wavefronts along the features x 2 along the tokens:
//   256 x 256: WN = 4, NI = 4, NJ = 8 (8 wavefronts of 64 features x 128 tokens);
//   288 x 192: WN = 4, NI = 3, NJ = 9 (8 wavefronts of 48 x 144) -- 9216 tokens x 3072 features are exactly 512 such
//              tiles, two rounds of 256 compute units, where 432 square tiles are 1.69;
//   192 x 192: WN = 4, NI = 3, NJ = 6 (8 wavefronts of 48 x 96; 2 - 5 % faster than 4 wavefronts of 96 x 96).
template <int NI, int NJ, int LAYOUT>
__global__ void __launch_bounds__(256, 1) qkv_gemm_direct_kernel(GemmArgs a) {
    constexpr int TM = 2 * NJ * 16, TN = 2 * NI * 16;             // tokens, features per tile
    constexpr int kXBytes = TM * BK * 2, kWBytes = TN * BK * 2;   // one operand tile of one K step
    constexpr int NMFMA = NI * NJ, NREADS = NI + NJ;              // per wavefront and half
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    constexpr uint32_t kWRing = kXSlots * kXBytes;          // the W slots follow the X slots
    const uint32_t K = (uint32_t)a.D;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wave_f = (wave & 1u) * (NI * 16u), wave_t = (wave >> 1) * (NJ * 16u);
    const TileWalk walk = tiles_of_block(a);
    uint32_t vt = walk.first;
    TileCoord tc = tile_at(a, vt);

    // Load i of this wavefront fills LDS rows (4 i + wave) * 8 .. + 8 of a tile (NJ loads for X, NI for W): lane -> row
    // lane >> 3, stored column lane & 7 (the swizzle of row 8 n + m depends on m and the parity of n, here the wavefront's).
    const uint32_t ld_row = wave * 8u + (lane >> 3), ld_col = ((lane & 7u) ^ swz(ld_row)) * 16u, ld_w_row = w_row_of(ld_row);
    const uint32_t ld_lds = lds0 + wave * 1024u;
    const unsigned char *xk, *wk;      // the operands' rows of the tile being loaded, at the K step that is loaded next
    uint32_t xoff[NJ], woff[NI];       // the lane's byte of each load; rows past the end re-read the last one and are never stored
    auto load_from = [&](const TileCoord& t) __attribute__((always_inline)) {
        xk = reinterpret_cast<const unsigned char*>(a.x + ((size_t)a.row_begin + t.m0) * K);
        wk = reinterpret_cast<const unsigned char*>(a.w[t.tensor] + (size_t)t.f0 * K);
#pragma unroll
        for (int i = 0; i < NJ; ++i) xoff[i] = min(32u * i + ld_row, (uint32_t)a.M - 1u - t.m0) * K * 2u + ld_col;
#pragma unroll
        for (int i = 0; i < NI; ++i) woff[i] = min(32u * i + ld_w_row, (uint32_t)a.D - 1u - t.f0) * K * 2u + ld_col;
    };
    load_from(tc);

    // MFMA operand layout: lane l holds 8 K elements (one 16-byte LDS column) of row l%16 of a 16-row fragment, lane
    // group l/16 the g-th eight of the instruction's 32.  Which column of the half a lane group takes is free as long as
    // W and X agree: groups 0, 1, 2, 3 take columns 0, 2, 1, 3, because a 128-bit LDS read serves lanes 8p .. 8p+7
    // together with lanes 32+8p .. 32+8p+7 (groups g and g+2), and rows 0 .. 7 of two columns share no bank only when
    // the columns differ in their lowest bit (measured: 4 conflict cycles per read with columns 0, 1, 2, 3).
    // Fragment addresses: row = wave offset + 16 i + (lane & 15); the swizzle depends on the lane only.
    const uint32_t frag_row = lane & 15u, frag_kg = ((lane >> 3) & 2u) | (lane >> 5);
    const uint32_t sw = swz(frag_row);
    const uint32_t frag_c[2] = {(frag_kg ^ sw) << 4, ((4u + frag_kg) ^ sw) << 4};
    const uint32_t x_frag = (wave_t + frag_row) * 128u;
    const uint32_t w_frag = kWRing + (wave_f + frag_row) * 128u;

    const uint32_t n_k = K / BK;   // >= 3 (the host sends shorter K to the fallback kernel)
    auto load_tile = [&](const unsigned char* base, const auto& off, uint32_t lds) __attribute__((always_inline)) {     // one operand's tile of one K step
        unrolled<(int)(sizeof(off) / sizeof(off[0]))>([&](auto i_c) __attribute__((always_inline)) {
            load_dest<4096 * decltype(i_c)::value>(lds);
            asm volatile("s_nop 0");
            load_to_lds(base, off[decltype(i_c)::value]);
        });
    };
    load_tile(xk, xoff, ld_lds);
    load_tile(wk, woff, ld_lds + kWRing);
    load_tile(xk + BK * 2, xoff, ld_lds + kXBytes);
    load_tile(wk + BK * 2, woff, ld_lds + kWRing + kWBytes);
    xk += 2 * BK * 2;
    wk += 2 * BK * 2;
    const bf16x8 zero = zero_fragment();
    unrolled<NI * NJ>([&](auto t_c) __attribute__((always_inline)) { clear_acc<4 * decltype(t_c)::value>(zero); });      // while the first loads are under way
    wait_loads<NI + NJ>();      // step 0 has landed; X1, W1 may still be in flight
    wave_barrier();

    // fragments of a half (32 K elements): one set is multiplied while the other is filled
    bf16x8 wf[2][NI], xf[2][NJ];
    auto read_frag = [&](bf16x8 (&w)[NI], bf16x8 (&x)[NJ], uint32_t xs, uint32_t ws, int kk, int r) {
        if (r < NI) w[r] = *reinterpret_cast<const bf16x8*>(smem + ws + w_frag + frag_c[kk] + r * 2048);
        else x[r - NI] = *reinterpret_cast<const bf16x8*>(smem + xs + x_frag + frag_c[kk] + (r - NI) * 2048);
    };
#pragma unroll
    for (int r = 0; r < NREADS; ++r) read_frag(wf[0], xf[0], 0, 0, 0, r);

    // One half: MFMA m multiplies W fragment i with X fragment j = m / NI of set CUR.  Between the MFMAs the NREADS fragments
    // of the next half are read into the other set and, with LOAD, this half's global -> LDS loads are issued (NJ of X in half
    // 0, NI of W in half 1), two instructions each.  These are dealt out evenly, about one to a gap: a wavefront issues one
    // instruction in four clocks and an MFMA takes sixteen, so more than three in a gap leave the matrix core idle, and with
    // one wavefront per SIMD nobody fills in.  The scalar bookkeeping of a step sits in gaps of its own for the same reason
    // (behind the last MFMA, with the branch, it cost 6 % of the loop's clocks).  After MFMA kBarrierAt of half 0 the wavefront
    // waits for its outstanding LDS reads and for all but its NJ youngest loads (LOAD; else all) and meets the others.
    // sched_barrier(0) keeps the order.
    //
    // K step kt: X in the ring slot at byte x_read, W in the one at byte w_read.  X of step kt+2 is issued during half 0 (into
    // the X slot x_load that step kt-1 used), W of step kt+2 during half 1 (into the W slot of step kt itself: behind this
    // step's barrier every wavefront has its fragments of step kt in registers).  At the barrier the loads in flight, oldest
    // first, are X(kt+1), W(kt+1), X(kt+2): the last may stay.
    static_assert(kXSlots == 3 && kWSlots == 2, "the slots below");
    uint32_t x_read = 0, x_next = kXBytes, x_load = 2 * kXBytes, w_read = 0;
    constexpr int kSpread = NMFMA >= 32 ? NMFMA - 16 : NMFMA >= 16 ? NMFMA - 6 : NMFMA;      // the gaps used for reads and loads
    constexpr int kBarrierAt = NMFMA >= 32 ? NMFMA - 8 : NMFMA - 1;
    constexpr int kTurnAt = NMFMA >= 32 ? NMFMA - 12 : NMFMA - 5;                            // and for the ring's turn
    static_assert(kTurnAt >= 0 && kTurnAt + 4 < NMFMA, "five gaps");
    auto half = [&](auto cur_c, auto load_c) __attribute__((always_inline)) {
        constexpr int CUR = decltype(cur_c)::value;
        constexpr bool LOAD = decltype(load_c)::value;
        constexpr int N_LOADS = !LOAD ? 0 : CUR == 0 ? NJ : NI, OPS = NREADS + 2 * N_LOADS;
        const uint32_t xs_n = CUR == 0 ? x_read : x_next, ws_n = CUR == 0 ? w_read : w_read ^ kWBytes;
        const uint32_t lds_l = CUR == 0 ? ld_lds + x_load : ld_lds + kWRing + w_read;
        uint32_t turning;
        unrolled<NMFMA>([&](auto m_c) __attribute__((always_inline)) {
            constexpr int m = decltype(m_c)::value;
            constexpr int q = m % NI, j = m / NI;                 // q-th MFMA of token tile j
            constexpr int i = (j & 1) ? NI - 1 - q : q;           // W fragments up, then down: one operand is kept at every turn
            mfma_acc<4 * (i * NJ + j)>(wf[CUR][i], xf[CUR][j]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (m < kSpread) {
                unrolled<(m + 1) * OPS / kSpread - m * OPS / kSpread>([&](auto t_c) __attribute__((always_inline)) {
                    constexpr int t = m * OPS / kSpread + decltype(t_c)::value;
                    constexpr int l = t * 2 * N_LOADS / OPS;       // load instructions before operation t
                    if constexpr ((t + 1) * 2 * N_LOADS / OPS == l) read_frag(wf[CUR ^ 1], xf[CUR ^ 1], xs_n, ws_n, CUR ^ 1, t - l);
                    else if constexpr (l % 2 == 0) load_dest<4096 * (l / 2)>(lds_l);
                    else if constexpr (CUR == 0) load_to_lds(xk, xoff[l / 2]);
                    else load_to_lds(wk, woff[l / 2]);
                });
            }
            if constexpr (CUR == 0 && m == kBarrierAt) {
                wait_loads_and_lds<N_LOADS>();
                wave_barrier();
            }
            if constexpr (LOAD && CUR == 0 && m == kTurnAt) xk += BK * 2;
            if constexpr (LOAD && CUR == 1 && m == kTurnAt) wk += BK * 2;
            if constexpr (CUR == 1 && m == kTurnAt + 1) set_scalar(turning, x_read);
            if constexpr (CUR == 1 && m == kTurnAt + 2) set_scalar(x_read, x_next);
            if constexpr (CUR == 1 && m == kTurnAt + 3) set_scalar(x_next, x_load);
            if constexpr (CUR == 1 && m == kTurnAt + 4) {
                set_scalar(x_load, turning);
                w_read ^= kWBytes;
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // The ring keeps turning from tile to tile: the last two steps of a tile load the first two of the workgroup's next one, and
    // the last half reads that tile's first fragments, so between two tiles only the epilogue's instructions are exposed -- no
    // workgroup start, no first trip to memory.
    auto k_step = [&](auto load) __attribute__((always_inline)) {
        reserve_accumulators();
        mfma_operands_ready();      // (fragments are copied where the loops meet)
        half(std::integral_constant<int, 0>{}, load);
        half(std::integral_constant<int, 1>{}, load);
    };
    const std::true_type loading;
    for (;;) {
        if (n_k & 1u) k_step(loading);
        uint32_t pairs = n_k / 2u - 1u;      // n_k - 2 steps in all; two to a turn of the loop (a branch taken costs some 80 clocks)
        if (pairs > 0) {
#pragma unroll 1
            do {
                k_step(loading);
                k_step(loading);
            } while (--pairs > 0);
        }
        vt += walk.stride;
        const bool more = vt < walk.end;
        const TileCoord next = tile_at(a, more ? vt : walk.first);
        if (more) {
            load_from(next);
            k_step(loading);
            k_step(loading);
        } else {
            k_step(std::false_type{});
            k_step(std::false_type{});      // (its very last half reads fragments nobody multiplies)
        }
        mfma_results_ready();

        const GemmArgs& e = arguments_again();
        const uint32_t tok = tc.m0 + wave_t, feat = tc.f0 + wave_f;
        TileOut out;
        out.live_j = (int)min((uint32_t)NJ, tok < (uint32_t)e.M ? ((uint32_t)e.M - tok) / 16u : 0u);
        out.live_p = (int)min((uint32_t)NI / 2u, feat < (uint32_t)e.D ? ((uint32_t)e.D - feat) / 32u : 0u);
        out.n0 = (uint32_t)e.row_begin + tok;
        out.tl = lane & 15u;
        out.v8 = feat / 8u + (lane >> 4);
        uint16_t* y = e.y[tc.tensor];
        if constexpr (LAYOUT == OUT_FUSED || LAYOUT == OUT_FUSED_ANY) {
            uint16_t* y2 = e.y2[tc.tensor];
            // the X slot of the step just finished is free until the next tile's first half loads into it again
            unsigned char* spare = smem + x_load;
            if (e.gamma[tc.tensor]) {     // the same for the whole workgroup: its barriers are taken by all or by none
                store_normalised<NI, NJ, LAYOUT == OUT_FUSED>(e, out, e.gamma[tc.tensor], y, y2, reinterpret_cast<float*>(spare), wave);
            } else if (e.sel_prev && tc.tensor == 0) {     // V (the first tensor of the launch), flagged on its way out
                const uint32_t mine = store_both<NI, NJ, true>(e, out, y, y2);
                // the verdicts of the two wavefronts that share the tokens
                uint32_t* verdicts = reinterpret_cast<uint32_t*>(spare);
                if (lane == 0) verdicts[wave] = mine;
                __syncthreads();
                const uint32_t any = verdicts[wave & ~1u] | verdicts[wave | 1u];
                if ((wave & 1u) == 0 && (int)lane < out.live_j)
                    e.sel_flag_bytes[(size_t)(out.n0 / 16u + lane) * 16u + tc.f0 / (uint32_t)TN] = (uint8_t)((any >> lane) & 1u);
                __syncthreads();     // before anybody loads into the slot again
            } else {
                store_both<NI, NJ, false>(e, out, y, y2);
            }
        } else {
            store_plain<NI, NJ, LAYOUT>(e, out, y);
        }
        if (!more) return;
        tc = next;
    }
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


// A tile shape of the main kernel with its two epilogues and launch parameters.
struct TileKernel {
    int bm, bn, threads, lds;
    double penalty;               // measured per-flop cost against the 256 x 256 tile
    const void* entry[5];         // by OutLayout (the fused ones only for the shapes of whole 256-feature tiles)
};
template <int NI, int NJ>
TileKernel tile_kernel(double penalty) {
    return {2 * NJ * 16, 2 * NI * 16, 256, ring_lds_bytes(2 * NJ * 16, 2 * NI * 16), penalty,
            {(const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_SEQ>, (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_CHUNKS>,
             (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_HEADS>, nullptr, nullptr}};
}
// a shape for the fused call only (tiles 256 features wide: whole heads of 64, 128 or 256)
template <int NI, int NJ>
TileKernel fused_tile_kernel(double penalty) {
    return {2 * NJ * 16, 2 * NI * 16, 256, ring_lds_bytes(2 * NJ * 16, 2 * NI * 16), penalty,
            {nullptr, nullptr, nullptr, (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_FUSED>,
             (const void*)qkv_gemm_direct_kernel<NI, NJ, OUT_FUSED_ANY>}};
}

// The tile shapes of the main kernel, and which one a launch of M tokens x D features x n_tensors weights takes.
// 256 x 256 does the least operand traffic per flop; the others are taken when their tile count fills the compute
// units so much better that they win all the same.  Cost = rounds x tile area x a measured per-flop penalty, a round
// being one tile on every unit.  (Measured and left out: 224 x 256 equals 288 x 192 at 9216 tokens and nothing else
// gains from it; 160 x 192, 256 x 192 and 192 x 256 win a few percent at 2304 tokens only.)
// whole_heads: the shapes of the fused call, all 256 features wide (a head row must lie inside one tile); their
// penalties follow the same two ratios (operand bytes and fragment reads per flop) as the measured ones.
static const TileKernel* tile_shapes(bool whole_heads, int* count) {
    static const TileKernel shapes[] = {tile_kernel<8, 8>(1.0), tile_kernel<6, 9>(kPenalty288), tile_kernel<6, 6>(kPenalty192)};
    static const TileKernel fused[] = {fused_tile_kernel<8, 8>(1.0), fused_tile_kernel<8, 7>(1.035), fused_tile_kernel<8, 6>(1.08)};
    *count = 3;
    return whole_heads ? fused : shapes;
}

struct LaunchPlan {
    const TileKernel* pick;    // nullptr: the compute-unit count could not be read
    bool ring_kernel;          // false: the general kernel (K not a multiple of 64, or shorter than three steps)
    int32_t bm, bn, tiles_m, tiles_n_per_tensor, n_cu;
};

static LaunchPlan plan_launch(int32_t M, int32_t D, int32_t n_tensors, bool whole_heads) {
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
    p.pick = &shapes[0];
    static const int forced_tile = (int)tune_value("COCODIFF_GEMM_TILE", 0);     // tuning builds only
    double best = 0.0;
    for (int i = 0; i < n_shapes; ++i) {
        const TileKernel& t = shapes[i];
        const int64_t tiles = (int64_t)((M + t.bm - 1) / t.bm) * ((D + t.bn - 1) / t.bn) * n_tensors;
        const double cost = (double)((tiles + n_cu - 1) / n_cu) * t.bm * t.bn * t.penalty;
        if (forced_tile ? forced_tile == t.bm * 1000 + t.bn : (i == 0 || cost < best)) {
            p.pick = &t;
            best = cost;
        }
    }
    p.ring_kernel = D % BK == 0 && D >= 3 * BK;
    p.bm = p.ring_kernel ? p.pick->bm : BM;      // the general kernel has one tile shape
    p.bn = p.ring_kernel ? p.pick->bn : BM;
    p.tiles_m = (M + p.bm - 1) / p.bm;
    p.tiles_n_per_tensor = (D + p.bn - 1) / p.bn;
    return p;
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
    const LaunchPlan plan = plan_launch(a.M, a.D, a.n_tensors, layout == OUT_FUSED);
    if (!plan.pick) return fail(COCODIFF_ERR_HIP, "qkv_proj: cannot read the compute-unit count");
    if (layout == OUT_FUSED && !plan.ring_kernel)
        return fail(COCODIFF_ERR_SHAPE, "qkv_proj_fused: D (%d) must be a multiple of 64 and at least 192", a.D);
    const TileKernel* pick = plan.pick;
    const bool ring_kernel = plan.ring_kernel;
    a.bm = plan.bm;
    a.bn = plan.bn;
    a.tiles_m = plan.tiles_m;
    a.tiles_n_per_tensor = plan.tiles_n_per_tensor;
    const uint32_t n_tiles = (uint32_t)a.tiles_m * a.tiles_n_per_tensor * a.n_tensors;
    a.n_tiles = (int32_t)n_tiles;
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
    if (ring_kernel)
        le = hipLaunchKernel(pick->entry[layout == OUT_FUSED && !quad_pairs ? OUT_FUSED_ANY : layout], dim3(n_tiles < (uint32_t)plan.n_cu ? n_tiles : (uint32_t)plan.n_cu), dim3(pick->threads), kernel_args, pick->lds, st);
    else
        le = hipLaunchKernel(staged[layout], dim3(n_tiles), dim3(kStagedThreads), kernel_args, kLdsBytes, st);
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

// Flag records of the projection that flags V: 16 bytes per 16-token tile, one byte per 256-feature tile of V.
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
    const uint32_t parts = (uint32_t)(shape->D + 255) / 256u;        // bytes of a record that the projection wrote
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
    const LaunchPlan p = plan_launch(shape->rank_count * (shape->N / shape->P), shape->D, n_tensors, whole_heads != 0);
    if (!p.pick) return fail(COCODIFF_ERR_HIP, "qkv_proj_plan: cannot read the compute-unit count");
    if (tile_tokens) *tile_tokens = p.bm;
    if (tile_features) *tile_features = p.bn;
    if (n_tiles) *n_tiles = p.tiles_m * p.tiles_n_per_tensor * n_tensors;
    if (n_compute_units) *n_compute_units = p.n_cu;
    return COCODIFF_OK;
}
