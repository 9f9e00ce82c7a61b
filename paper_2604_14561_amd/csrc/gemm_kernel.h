// The projection's main kernel (see gemm.hip for the whole): a template over tile shape and output layout, instantiated one
// layout to a source file.
#pragma once

#include <type_traits>
#include <utility>

#include "internal.h"

namespace cocodiff {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int BK = 64;           // K elements per step
struct GemmArgs {
    const uint16_t* x;
    const uint16_t* w[3];
    uint16_t* y[3];
    int32_t n_tensors;
    int32_t row_begin, M;      // token rows [row_begin, row_begin + M)
    int32_t D;                 // features per tensor = K
    int32_t tiles_m, tiles_n_per_tensor, n_tiles;
    int32_t bm, bn;            // tile of the launch: tokens x features
    uint32_t workers;          // workgroups that walk tiles; those behind them fetch operands (fetch_operands), from this
    uint32_t fetch_from;       // column on
    uint32_t group;            // tile rows that are walked together (tile_at)
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
// OUT_CHUNKS_STREAMED, OUT_FUSED_STREAMED: the chunks, and the fused form's head-parallel V, streamed past the caches too (streams_outputs
// in gemm.hip says when; the chunks by tiles 256 and 128 features wide only).  Layouts of their own: a branch in the epilogue costs a launch of one round more than it gains (3600 x 1152
// 36.3 us without, 37.3 with, 35.5 so).
enum OutLayout { OUT_SEQ = 0, OUT_CHUNKS = 1, OUT_HEADS = 2, OUT_FUSED = 3, OUT_FUSED_ANY = 4, OUT_CHUNKS_STREAMED = 5, OUT_FUSED_STREAMED = 6 };
constexpr int kLayouts = 7;
constexpr bool is_fused(int layout) { return layout == OUT_FUSED || layout == OUT_FUSED_ANY || layout == OUT_FUSED_STREAMED; }
constexpr bool is_chunks(int layout) { return layout == OUT_CHUNKS || layout == OUT_CHUNKS_STREAMED; }

// [rows][64] bf16 tiles (128-byte rows): any 16 consecutive rows of one column land in 16 different
// 16-byte slots of the 256-byte bank span.
__device__ __forceinline__ uint32_t swz(uint32_t row) { return (row & 7u) ^ ((row >> 3) & 1u); }

struct TileCoord {
    uint32_t tensor, m0, f0;
};

// Tile `vt` of the launch: groups of a.group tile rows walked column by column, so that tiles with neighbouring numbers share
// rows of X and W.
__device__ __forceinline__ TileCoord tile_at(const GemmArgs& a, uint32_t vt) {
    const uint32_t tiles_n = (uint32_t)a.tiles_n_per_tensor * a.n_tensors;
    const uint32_t per_group = a.group * tiles_n;
    const uint32_t grp = vt / per_group;
    const uint32_t first_m = grp * a.group;
    const uint32_t rows_here = min((uint32_t)a.tiles_m - first_m, a.group);
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
    return {begin + (blockIdx.x >> 3), begin + per + (xcd < rem ? 1u : 0u), (a.workers >> 3) + (xcd < (a.workers & 7u) ? 1u : 0u)};
}

// The accumulators live in the accumulation registers a0 .. a255 by number, and the compiler does not know them: accumulator
// tile (i, j) is a[4 (i NJ + j)] and the three behind it.  (Left to the compiler, it moves accumulators between the two
// register files and to scratch memory -- at 256 of them the loops over K steps and tiles carry 128 moves each way per step.)
// reserve_accumulators in every K step and every token tile of the epilogue tells it that all of them change, so it keeps
// nothing of its own there from one of these places to the next.  That does not forbid a copy that lives between two of them: the
// build reads the kernels' assembly and fails on any use of these registers that is not written here (build.py,
// accumulator_accesses).  The waits that these instructions need are in the code too: an MFMA
// result is read only behind mfma_results_ready(), and many instructions lie between clearing an accumulator and the next MFMA
// on it.
#define COCODIFF_ACC_0_63 \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", \
    "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", \
    "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", \
    "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63"
#define COCODIFF_ACC_64_255 \
    "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", \
    "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", \
    "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", \
    "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", \
    "a127", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", \
    "a141", "a142", "a143", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", \
    "a155", "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", \
    "a169", "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", \
    "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", \
    "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", \
    "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", \
    "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", \
    "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", \
    "a253", "a254", "a255"
template <int COUNT>
__device__ __forceinline__ void reserve_accumulators() {
    if constexpr (COUNT <= 64) asm volatile("" ::: COCODIFF_ACC_0_63);
    else asm volatile("" ::: COCODIFF_ACC_0_63, COCODIFF_ACC_64_255);
}
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
// the next tile's operands meanwhile.  A store instruction writes 64 consecutive bytes of sixteen tokens (the fused form
// exchanges vectors between lanes first and writes whole lines of eight, see pair_lines).
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

// Whole lines for streamed stores.  A store of one vector per lane writes 64 consecutive bytes of sixteen tokens: half a line each,
// its other half a vector later.  Streamed past the caches such halves cost: 64 x 72 tokens, 16 heads of 64, 84 tiles of V
// and 168 of Q and K in one round, all storing at once: the fused epilogue took 24.9 k clocks of the tile's 61 k, 20.9 k with
// whole lines; the call 41.4 -> 38.1 us, at 144 x 144 tokens, 24 heads of 128, 968 -> 916 us.
// pair_lines exchanges the vectors of features 32 p .. (`a`) and 32 (p + 1) .. (`b`), p even, between the lanes of tokens t and
// t + 8 of a token tile: `a` becomes the line of tokens 0 .. 7, the upper half of it in the lanes of tokens 8 .. 15, and `b` that
// of tokens 8 .. 15.  paired() moves a lane's destinations along.
__device__ __forceinline__ void pair_lines(vec16& a, vec16& b) {
    constexpr int ROW_ROR_8 = 0x128;      // from the lane 8 further in the same row of 16; written in the upper / lower half row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int x = (int)a[i], y = (int)b[i];
        a[i] = (uint32_t)__builtin_amdgcn_update_dpp(x, y, ROW_ROR_8, 0xf, 0xc, false);
        b[i] = (uint32_t)__builtin_amdgcn_update_dpp(y, x, ROW_ROR_8, 0xf, 0x3, false);
    }
}
template <int NP>
__device__ __forceinline__ Dest<NP> paired(Dest<NP> t, uint32_t tl, uint32_t row) {      // row: vectors from one token to the next
    static_assert(NP % 2 == 0, "feature groups in pairs");
#pragma unroll
    for (int p = 0; p < NP; p += 2) {
        if (tl >= 8u) t.lane[p] = t.lane[p + 1] - (size_t)8u * row;
        t.lane[p + 1] = t.lane[p] + (size_t)8u * row;
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
__device__ __forceinline__ void peek_acc(float (&x)[8]) {
    unrolled<8>([&](auto e_c) __attribute__((always_inline)) {
        constexpr int e = decltype(e_c)::value;
        x[e] = read_acc<4 * ((2 * P + e / 4) * NJ + J) + e % 4>();
    });
}
// The same, and the accumulators are cleared for the workgroup's next tile.
template <int NJ, int P, int J>
__device__ __forceinline__ void take_acc(float (&x)[8], const bf16x8& zero) {
    peek_acc<NJ, P, J>(x);
    clear_acc<4 * (2 * P * NJ + J)>(zero);
    clear_acc<4 * ((2 * P + 1) * NJ + J)>(zero);
}
// f(token tile, a constant) for those that exist; the others' accumulators are cleared here.
template <int NI, int NJ, typename F>
__device__ __forceinline__ void for_token_tiles(const TileOut& t, const bf16x8& zero, F&& f) {
    unrolled<NJ>([&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        reserve_accumulators<4 * NI * NJ>();
        if (j < t.live_j)
            f(j_c);
        else
            unrolled<NI>([&](auto i_c) __attribute__((always_inline)) { clear_acc<4 * (decltype(i_c)::value * NJ + j)>(zero); });
    });
}
// The vectors of one token tile to y.  (D is a multiple of 64: where a wavefront's groups of 32 features come in pairs, so do
// the missing ones.)
template <bool NT, int NP>
__device__ __forceinline__ void store_groups(vec16* __restrict__ y, const Dest<NP>& to, const vec16 (&v)[NP], int live_p) {
#pragma unroll
    for (int p = 0; p < NP; p += NP % 2 ? 1 : 2) {
        if (p < live_p) {
            st_vec<NT>(y + to.lane[p], v[p]);
            if (NP % 2 == 0) st_vec<NT>(y + to.lane[p + 1], v[p + 1]);
        }
    }
}

// Sum over the four lanes that hold one token's features (lanes l, l+16, l+32, l+48), in all four.
__device__ __forceinline__ float sum_of_token(float s) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The sum of the two halves of a head, each as sum_of_token forms it, in all four lanes: the exchange between the rows of 16 lanes leaves
// `first` in the even and `second` in the odd ones, so one more exchange does instead of two.
__device__ __forceinline__ float sum_of_halves(float first, float second) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(first), __float_as_uint(second), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    const float t = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

// Stores.  Cache policy: what a kernel of the same step reads next stays cached -- [N][D], the head-parallel V (the
// selection reads it), and the exchange buffer of cocodiff_qkv_proj_pack (its unpack follows) -- but for the STREAMED layouts.
// In the fused call nothing on this GPU reads the exchange buffers (they are what the all-to-all would send) or, within the
// step, the head-parallel Q and K: streamed past the caches they leave nothing dirty in L2 to be written back under the next
// round's loads.
template <int NI, int NJ, int LAYOUT>
__device__ __forceinline__ void store_plain(const GemmArgs& a, const TileOut& t, uint16_t* __restrict__ Y) {
    constexpr int NP = NI / 2;
    constexpr bool STREAM = LAYOUT == OUT_CHUNKS_STREAMED;
    static_assert(!STREAM || NP % 2 == 0, "whole lines: feature groups in pairs");
    Dest<NP> to = LAYOUT == OUT_SEQ ? dest_seq<NP>(a, t.v8, t.tl) : is_chunks(LAYOUT) ? dest_chunks<NP>(a, t.v8, t.tl) : dest_heads<NP>(a, t.v8, t.tl);
    if constexpr (STREAM) to = paired(to, t.tl, a.row8);
    ChunkWalk chunk(a, t.n0);
    const uint32_t row = LAYOUT == OUT_SEQ ? (uint32_t)a.D / 8u : a.d8;
    vec16* y = reinterpret_cast<vec16*>(Y) + (is_chunks(LAYOUT) ? 0 : (size_t)t.n0 * row);
    const bf16x8 zero = zero_fragment();
    for_token_tiles<NI, NJ>(t, zero, [&](auto j_c) __attribute__((always_inline)) {
        vec16 v[NP];
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            float x[8];
            take_acc<NJ, decltype(p_c)::value, decltype(j_c)::value>(x, zero);
            v[decltype(p_c)::value] = pack_vec(x);
        });
        if constexpr (STREAM) {
#pragma unroll
            for (int p = 0; p < NP; p += 2) pair_lines(v[p], v[p + 1]);
        }
        if (is_chunks(LAYOUT)) {
            store_groups<STREAM>(y + chunk.at, to, v, t.live_p);
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
template <int NI, int NJ, bool SELECT, bool STREAM>
__device__ __forceinline__ uint32_t store_both(const GemmArgs& a, const TileOut& t, uint16_t* __restrict__ Y, uint16_t* __restrict__ Y2) {
    // (fetched 7 token tiles ahead: 32 x 48 tokens, 24 heads of 128, the call 81.6 us with 5, 79.1 so)
    constexpr int NP = NI / 2, AHEAD = NJ < 7 ? NJ : 7;
    const Dest<NP> to_c = paired(dest_chunks<NP>(a, t.v8, t.tl), t.tl, a.row8), to_h = paired(dest_heads<NP>(a, t.v8, t.tl), t.tl, a.d8);
    ChunkWalk chunk(a, t.n0);
    const size_t at0 = (size_t)t.n0 * a.d8, step = (size_t)16u * a.d8;
    vec16 *yc = reinterpret_cast<vec16*>(Y), *yh = reinterpret_cast<vec16*>(Y2) + at0;
    const vec16* yp = reinterpret_cast<const vec16*>(a.sel_prev) + at0;
    // The previous V's lines are loaded whole, laid out as the vectors that they are compared with.  Streamed loads, but cached ones
    // where every unit has one tile and all of V is read at once, behind the K loops: the whole call 39.8 us streamed and 38.1 cached
    // at 4608 x 1024, 41.2 and 40.0 at 3600 x 1152, 48.3 and 46.8 at 3072 x 1536; 80.3 and 81.4 at 1536 x 3072.
    const bool one_round = (uint32_t)a.n_tiles <= a.workers;
    vec16 prev[AHEAD + 1][NP];
    auto fetch = [&](int j) __attribute__((always_inline)) {
        if (SELECT && j < t.live_j) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (p < t.live_p) prev[j % (AHEAD + 1)][p] = one_round ? yp[step * j + to_h.lane[p]] : ld_nt(yp + step * j + to_h.lane[p]);
        }
    };
#pragma unroll
    for (int j = 0; j < AHEAD && j < NJ; ++j) fetch(j);
    uint32_t verdict = 0, ties = 0;
    const bf16x8 zero = zero_fragment();
    for_token_tiles<NI, NJ>(t, zero, [&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        if constexpr (j + AHEAD < NJ) fetch(j + AHEAD);
        vec16 v[NP];
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            float x[8];
            take_acc<NJ, decltype(p_c)::value, j>(x, zero);
            v[decltype(p_c)::value] = pack_vec(x);
        });
#pragma unroll
        for (int p = 0; p < NP; p += 2) pair_lines(v[p], v[p + 1]);
        if (Y) store_groups<true>(yc + chunk.at, to_c, v, t.live_p);
        if (Y2) store_groups<STREAM>(yh, to_h, v, t.live_p);
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
#pragma unroll
            for (int p = 0; p < NP; ++p)      // (every lane what it stored itself)
                if (p < t.live_p) changed |= vec_changed_double(now[to_h.lane[p]], yp[step * j + to_h.lane[p]], a.sel_th.tau);
            verdict |= (__ballot(changed) != 0 ? 1u : 0u) << j;
        }
    }
    return verdict;
}

// RMSNorm over every head row and RoPE on the fp32 accumulators, in the arithmetic order of the stand-alone norm + RoPE
// kernel (x * rinv * gamma, then the rotation) -- but on the unrounded projection, so Q and K are rounded to bf16 once
// instead of twice -- and out to both destinations.
// HEAD = d.  A wavefront holds 16 NI features of its tokens: one or two whole heads, or half of one, whose sums of squares the
// two wavefronts exchange through `xch` (LDS, [wavefront][token]; two workgroup barriers, the second so that
// nobody overwrites what the other still reads).
// A head of 128 is summed in halves of 64 features also where one wavefront holds it: the bits of Q and K do not depend on the
// tile, so a call that flags V, or takes a range of the ranks, gives those of the call it stands for.
// Nothing else runs on the unit meanwhile, so this stage's instructions are exposed (where all units end together its stores take
// longer still): the token's grid coordinates are divided out once, for token tile 0, and then stepped as table row offsets: 16 tokens further is a.row_step16[] further in
// mixed radix, with carries (the absent axes of a one- or two-axis grid are grids of one cell: they never carry).  The
// (cos, sin) values of a token tile are fetched from the table (L1 / L2) while its sums of squares are formed.
// QUADS: every axis has a multiple of four pairs, so the four pairs of a vector are 32 consecutive bytes of a table row.
template <int NI, int NJ, bool QUADS, int HEAD>
__device__ __forceinline__ void store_normalised(const GemmArgs& a, const TileOut& t, const uint16_t* __restrict__ gamma, uint16_t* __restrict__ Y,
                                                 uint16_t* __restrict__ Y2, float* xch, uint32_t wave) {
    constexpr int NP = NI / 2;
    constexpr int WF = NI * 16, HEADS = WF >= HEAD ? WF / HEAD : 1;      // features of a wavefront; whole heads among them
    constexpr bool WIDE = HEAD > WF;                                     // a head of two wavefronts
    constexpr int SUMS = HEAD == 128 && !WIDE ? 2 * HEADS : HEADS;
    static_assert((WF == 64 || WF == 128) && (HEAD == 64 || HEAD == 128 || HEAD == 256) && HEAD <= 2 * WF, "heads per tile");
    if (WIDE) {
        unrolled<NJ>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value;
            reserve_accumulators<4 * NI * NJ>();
            float s = 0.f;
            unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
                float x[8];
                peek_acc<NJ, decltype(p_c)::value, j>(x);
#pragma unroll
                for (int e = 0; e < 8; ++e) s += x[e] * x[e];
            });
            s = sum_of_token(s);
            xch[wave * (NJ * 16) + 16 * j + t.tl] = s;      // (four lanes, one value)
        });
        __syncthreads();
    }

    // the lane's rotary pairs of feature group p (4; without QUADS their axes may differ): which axis' row, as masks, and the
    // float offset from that row's start
    constexpr int NQ = QUADS ? 1 : 4;
    const uint32_t p0 = (uint32_t)a.rope.pairs[0], p01 = p0 + (uint32_t)a.rope.pairs[1];
    uint32_t on_1[NP][NQ], on_2[NP][NQ], col[NP][NQ];
    vec16 g[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t fh = (8u * (t.v8 + 4u * p)) & (HEAD - 1u);      // the vector's first feature inside its head
        g[p] = *reinterpret_cast<const vec16*>(gamma + fh);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t pr = fh / 2u + q;
            on_2[p][q] = a.rope.n_axes > 2 && pr >= p01 ? ~0u : 0u;
            on_1[p][q] = a.rope.n_axes > 1 && pr >= p0 ? ~on_2[p][q] : 0u;
            col[p][q] = 2u * pr - (on_2[p][q] & (2u * p01)) - (on_1[p][q] & (2u * p0));
        }
    }
    // float offsets of the token's row in each axis' table, for this lane's token of the current token tile
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
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t row = (row_a[2] & on_2[p][q]) | (row_a[1] & on_1[p][q]) | (row_a[0] & ~(on_1[p][q] | on_2[p][q]));
                const float* at = cs_table + (row + col[p][q]);
                if (QUADS) {
                    const float4 lo = *reinterpret_cast<const float4*>(at), hi = *reinterpret_cast<const float4*>(at + 4);
                    to[p][0] = lo.x; to[p][1] = lo.y; to[p][2] = lo.z; to[p][3] = lo.w;
                    to[p][4] = hi.x; to[p][5] = hi.y; to[p][6] = hi.z; to[p][7] = hi.w;
                } else {
                    const float2 c = *reinterpret_cast<const float2*>(at);
                    to[p][2 * q] = c.x;
                    to[p][2 * q + 1] = c.y;
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

    const Dest<NP> to_c = paired(dest_chunks<NP>(a, t.v8, t.tl), t.tl, a.row8), to_h = paired(dest_heads<NP>(a, t.v8, t.tl), t.tl, a.d8);
    ChunkWalk chunk(a, t.n0);
    vec16 *yc = reinterpret_cast<vec16*>(Y), *yh = reinterpret_cast<vec16*>(Y2) + (size_t)t.n0 * a.d8;
    const bf16x8 zero = zero_fragment();
    for_token_tiles<NI, NJ>(t, zero, [&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        float cs[NP][8];
        load_cs(cs);
        next_token_tile();
        float x[NP][8], s[SUMS] = {};
        unrolled<NP>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            take_acc<NJ, p, j>(x[p], zero);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[p * SUMS / NP] += x[p][e] * x[p][e];
        });
        float rinv[HEADS];
#pragma unroll
        for (int u = 0; u < HEADS; ++u) {
            const float ss = WIDE ? xch[(wave & ~1u) * (NJ * 16) + 16 * j + t.tl] + xch[(wave | 1u) * (NJ * 16) + 16 * j + t.tl]
                             : SUMS > HEADS ? sum_of_halves(s[0], s[SUMS - 1]) : sum_of_token(s[u]);
            rinv[u] = 1.0f / sqrtf(ss * a.inv_d + a.eps);
        }
        vec16 v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t gw[4] = {g[p].x, g[p].y, g[p].z, g[p].w};
            float o[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float ev = x[p][2 * q] * rinv[p * HEADS / NP] * bf16_lo(gw[q]);
                const float od = x[p][2 * q + 1] * rinv[p * HEADS / NP] * bf16_hi(gw[q]);
                o[2 * q] = ev * cs[p][2 * q] - od * cs[p][2 * q + 1];
                o[2 * q + 1] = ev * cs[p][2 * q + 1] + od * cs[p][2 * q];
            }
            v[p] = pack_vec(o);
        }
#pragma unroll
        for (int p = 0; p < NP; p += 2) pair_lines(v[p], v[p + 1]);
        if (Y) store_groups<true>(yc + chunk.at, to_c, v, t.live_p);
        if (Y2) store_groups<true>(yh, to_h, v, t.live_p);
        chunk.next(a);
        yh += (size_t)16u * a.d8;
    });
    if (WIDE) __syncthreads();      // before anybody loads into the exchange's slot again
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
// Main kernel.  Four wavefronts, two along the features x two along the tokens, one per SIMD; a wavefront's tile is 16 NI
// features x 16 NJ tokens.  (The 256 x 256 tile on eight wavefronts of 64 x 128, two per SIMD, reads half as much again from
// LDS per flop and issues half as much again beside its MFMAs; one launch at 16384 x 3072 x 3072: 223 us, 1.39 PFLOP/s, the
// matrix cores busy 69 % of its clocks; this form 201 us, 1.54 PFLOP/s, 77 %.)
// A step's X tile and W tile travel through two rings in LDS.  Loads run kAhead steps ahead: kAhead + 1 slots for X tiles and
// kAhead for W tiles -- 160 KB for a 256 x 256 tile with two steps, as many as fit (up to four) for smaller ones, whose steps
// are shorter than a trip to memory (128 x 128, 48 steps, fewer tiles than units: 25 us with two steps ahead).
// A K step is two halves of 32 K elements, one v_mfma_f32_16x16x32_bf16 per 16 x 16 output tile and half.  In step kt a
// wavefront multiplies half 0 while reading the fragments of half 1, waits until step kt+1 has landed (its own loads; the
// barrier covers the other wavefronts'), then multiplies half 1 while reading half 0 of step kt+1.  After that barrier every
// wavefront has its fragments of step kt in registers, so W of step kt+kAhead goes into the W slot of step kt (from there on,
// through half 1) and X of step kt+1+kAhead into its X slot (during half 0 of step kt+1).
// ---------------------------------------------------------------------------------------------
constexpr int kMaxLds = 160 * 1024;
constexpr int ring_lds(int bm, int bn, int ahead) { return ((ahead + 1) * bm + ahead * bn) * BK * 2; }
constexpr int steps_ahead(int bm, int bn) { return ring_lds(bm, bn, 4) <= kMaxLds ? 4 : ring_lds(bm, bn, 3) <= kMaxLds ? 3 : 2; }
constexpr int ring_lds_bytes(int bm, int bn) { return ring_lds(bm, bn, steps_ahead(bm, bn)); }
// Workgroups that share a compute unit: two where the rings fit twice (64 x 64 and 32 x 64 tiles); the kernel's launch bounds then
// keep a wavefront to the 256 registers that leaves it (138 and 122 taken).
constexpr int workgroups_per_unit(int ni, int nj) { return 2 * ring_lds_bytes(32 * nj, 32 * ni) <= kMaxLds ? 2 : 1; }

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

// What units without a tile do in a launch of one round: read a word of each line of the launch's operands, from column a.fetch_from on
// in the order in which the K loops come to them.  A K step's loads are a few steps ahead, less than a trip to memory takes; so
// the tiles find their operands in the last-level cache.  (Streamed loads leave nothing there.)
// 64 units of 256 without a tile and 16, cold: 768 tokens of 9216, 3072 features, one weight and two with norm and rotation, and the
// other calls of that rank, 72.8 -> 67.7 us; the latter launch alone 38.4 -> 31.9, 29.4 with everything on chip.
// By XCD, each fetching what its own units read into its L2, is slower than none: three to seven times the lines, and a unit
// takes some 37 bytes a clock whoever it reads for.
// Where the operands are on chip already -- the same weights again, with less than the last-level cache in between -- fetching takes
// bandwidth from the tiles for nothing.  Whole layers in one call (11, 256 .. 2304 tokens x 1408 .. 3072 features), without and with it: all on
// chip 1.4 % more (3 to 5 % at most), around the cache's size 13 % less, from memory 12 % less.  A workgroup cannot tell which it is: asked for 128
// lines, of which it leaves if all come within 0.42 us, 1.0, -9 and -12 %, within 0.50 us 0.3, -4 and -12 %; a load takes 0.28 to 0.44 us
// from the last-level cache under load, and 0.44 to 0.5 from memory that has little else to do, while a tenth of the lines missing makes the
// tiles wait at every step.  (Votes of a workgroup's wavefronts and samples spread over all rows: between the same ends.  Resting 512 to
// 2048 clocks between batches of four loads: the same on chip, 0 to 5 % more from memory.)
constexpr uint32_t kFetchLines = 8;      // a column: 8 lines of every row, 8 K steps
__device__ __forceinline__ void fetch_operands(const GemmArgs& a) {
    constexpr uint32_t kLine = BK * 2, kRows = 64 / kFetchLines, kInFlight = 16;
    const uint32_t K = (uint32_t)a.D, row_lines = K * 2u / kLine, rows = (uint32_t)a.M + (uint32_t)a.n_tensors * K;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = (gridDim.x - a.workers) * 4u;
    const uint32_t blocks = (rows + kRows - 1u) / kRows, columns = (row_lines + kFetchLines - 1u) / kFetchLines;
    uint32_t block = (blockIdx.x - a.workers) * 4u + wave, column = a.fetch_from;      // a load: one column of kRows rows
    while (column < columns) {
        uint32_t got[kInFlight] = {};
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u) {
            while (block >= blocks) {
                block -= blocks;
                ++column;
            }
            const uint32_t r = min(block * kRows + lane / kFetchLines, rows - 1u);
            const uint32_t line = min(min(column, columns - 1u) * kFetchLines + lane % kFetchLines, row_lines - 1u);
            const uint32_t f = r - (uint32_t)a.M;
            const uint16_t* row = r < (uint32_t)a.M ? a.x + ((size_t)a.row_begin + r) * K
                                  : f < K           ? a.w[0] + (size_t)f * K
                                  : f < 2u * K      ? a.w[1] + (size_t)(f - K) * K
                                                    : a.w[2] + (size_t)(f - 2u * K) * K;
            if (column < columns) got[u] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(row) + line * kLine);
            block += waves;
        }
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u) asm volatile("" ::"v"(got[u]));
    }
}

// Scalar steps of the K loop, kept where they are written.
__device__ __forceinline__ void set_scalar(uint32_t& to, uint32_t from) { asm volatile("s_mov_b32 %0, %1" : "=s"(to) : "s"(from)); }

// The workgroup's barrier without the fence of __syncthreads() (which drains the LDS reads in flight): what has to have
// completed is waited for in front of it.
__device__ __forceinline__ void wave_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Tile = 32 NJ tokens x 32 NI features: NI = NJ = 8 is 256 x 256, NI = 6, NJ = 9 is 288 x 192 -- 9216 tokens x 3072 features are
// exactly 512 of those, two rounds of 256 compute units, where 432 square tiles are 1.69.
template <int NI, int NJ, int LAYOUT>
__global__ void __launch_bounds__(256, workgroups_per_unit(NI, NJ)) qkv_gemm_direct_kernel(GemmArgs a) {
    fetch_arguments<sizeof(GemmArgs)>();
    if (blockIdx.x >= a.workers) {
        fetch_operands(a);
        return;
    }
    constexpr int TM = 2 * NJ * 16, TN = 2 * NI * 16;             // tokens, features per tile
    constexpr int kXBytes = TM * BK * 2, kWBytes = TN * BK * 2;   // one operand tile of one K step
    constexpr int NMFMA = NI * NJ, NREADS = NI + NJ;              // per wavefront and half
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    constexpr int kAhead = steps_ahead(TM, TN);
    constexpr uint32_t kWRing = (kAhead + 1) * kXBytes;      // the W slots follow the X slots
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

    const uint32_t n_k = K / BK;   // >= kAhead (the host's choice of a tile sees to it)
    auto load_tile = [&](const unsigned char* base, const auto& off, uint32_t lds) __attribute__((always_inline)) {     // one operand's tile of one K step
        unrolled<(int)(sizeof(off) / sizeof(off[0]))>([&](auto i_c) __attribute__((always_inline)) {
            load_dest<4096 * decltype(i_c)::value>(lds);
            asm volatile("s_nop 0");
            load_to_lds(base, off[decltype(i_c)::value]);
        });
    };
    unrolled<kAhead>([&](auto s_c) __attribute__((always_inline)) {
        constexpr uint32_t s = decltype(s_c)::value;
        load_tile(xk, xoff, ld_lds + s * kXBytes);
        load_tile(wk, woff, ld_lds + kWRing + s * kWBytes);
        xk += BK * 2;
        wk += BK * 2;
    });
    const bf16x8 zero = zero_fragment();
    unrolled<NI * NJ>([&](auto t_c) __attribute__((always_inline)) { clear_acc<4 * decltype(t_c)::value>(zero); });      // while the first loads are under way
    wait_loads<(kAhead - 1) * (NI + NJ)>();      // step 0 has landed
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
    // of the next half are read into the other set and, but for the last steps, this half's global -> LDS loads are issued (NJ of X in half
    // 0, NI of W in half 1), two instructions each.  These are dealt out evenly, about one to a gap: a wavefront issues one
    // instruction in four clocks and an MFMA takes sixteen, so more than three in a gap leave the matrix core idle, and with
    // one wavefront per SIMD nobody fills in.  The scalar bookkeeping of a step sits in gaps of its own for the same reason
    // (behind the last MFMA, with the branch, it cost 6 % of the loop's clocks).  After MFMA kBarrierAt of half 0 the wavefront
    // waits for its outstanding LDS reads and for the loads of step kt+1 and meets the others.
    // sched_barrier(0) keeps the order.
    //
    // K step kt: X in the ring slot at byte x_read, W in the one at byte w_read.  X of step kt+kAhead is issued during half 0
    // (into the X slot x_load that step kt-1 used), W of step kt+kAhead from the barrier on and through half 1 (into the W slot of
    // step kt itself).  At the barrier what is younger than step kt+1's loads may stay in flight: the loads of kAhead - 2 whole
    // steps and the X loads of one more; in the last steps, which load nothing (TAIL = how many steps follow), those of TAIL - 1
    // steps.
    uint32_t x_read = 0, x_next = kXBytes, x_load = kAhead * kXBytes, w_read = 0, w_next = kWBytes;
    constexpr int kSpread = NMFMA >= 32 ? NMFMA - 16 : NMFMA >= 16 ? NMFMA - 6 : NMFMA;      // the gaps used for reads and loads
    constexpr int kBarrierAt = NMFMA >= 32 ? NMFMA - 8 : NMFMA - 1;
    // W's first loads of a step go out behind the barrier already, which frees their slot, an instruction to a gap: of all loads W's have
    // the shortest way to go, from there to the next step's barrier.  (Weights that come from memory, 24 heads of 128, whole calls
    // with W's loads dealt out over half 1 and so: 48 x 48 tokens 122.1 and 118.9 us, 16 x 60 x 104 4335 and 4275; 96 x 96
    // 407.7 and 404.3; others within 0.3 %.)
    constexpr int kEarly = (NMFMA - 1 - kBarrierAt) / 2;
    constexpr int kTurnAt = NMFMA >= 32 ? NMFMA - 12 : NMFMA > 5 ? NMFMA - 5 : 0;            // and, from there on, for the ring's turn
    constexpr auto turn_at = [](int n) { return kTurnAt + n < NMFMA ? kTurnAt + n : NMFMA - 1; };
    constexpr int kAdvanceAt = kTurnAt >= kSpread ? kTurnAt : NMFMA - 1;      // the operand pointers move on: behind the half's last load
    static_assert(kAdvanceAt >= kSpread - 1, "the loads of a half use the pointers of that half");
    auto half = [&](auto cur_c, auto tail_c, auto read_c) __attribute__((always_inline)) {
        constexpr int CUR = decltype(cur_c)::value, TAIL = decltype(tail_c)::value;
        constexpr bool READ = decltype(read_c)::value;
        constexpr bool LOAD = TAIL < 0;
        constexpr int EARLY = CUR == 0 ? 0 : kEarly, N_LOADS = !LOAD ? 0 : CUR == 0 ? NJ : NI - kEarly, OPS = (READ ? NREADS : 0) + 2 * N_LOADS;
        constexpr int IN_FLIGHT = LOAD ? (kAhead - 1) * NJ + (kAhead - 2) * NI : TAIL > 1 ? (TAIL - 1) * (NI + NJ) : 0;
        const uint32_t xs_n = CUR == 0 ? x_read : x_next, ws_n = CUR == 0 ? w_read : w_next;
        const uint32_t lds_l = CUR == 0 ? ld_lds + x_load : ld_lds + kWRing + w_read;
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
                    else if constexpr (l % 2 == 0) load_dest<4096 * (EARLY + l / 2)>(lds_l);
                    else {
                        // (its M0 is set by the operation before: where that one is in the same gap, no MFMA lies between)
                        if constexpr (decltype(t_c)::value > 0) asm volatile("s_nop 0");
                        if constexpr (CUR == 0) load_to_lds(xk, xoff[l / 2]);
                        else load_to_lds(wk, woff[EARLY + l / 2]);
                    }
                });
            }
            if constexpr (CUR == 0 && m == kBarrierAt) {
                wait_loads_and_lds<IN_FLIGHT>();
                wave_barrier();
            }
            if constexpr (LOAD && CUR == 0 && m > kBarrierAt && (m - kBarrierAt - 1) / 2 < kEarly) {
                constexpr int l = (m - kBarrierAt - 1) / 2;
                if constexpr ((m - kBarrierAt) % 2 == 1) load_dest<4096 * l>(ld_lds + kWRing + w_read);
                else load_to_lds(wk, woff[l]);
            }
            if constexpr (LOAD && CUR == 0 && m == kAdvanceAt) xk += BK * 2;
            if constexpr (LOAD && CUR == 1 && m == kAdvanceAt) wk += BK * 2;
            if constexpr (CUR == 1 && m == turn_at(1)) set_scalar(x_load, x_read);
            if constexpr (CUR == 1 && m == turn_at(2)) set_scalar(x_read, x_next);
            if constexpr (CUR == 1 && m == turn_at(3)) {
                x_next = x_next == kAhead * kXBytes ? 0u : x_next + kXBytes;
                asm volatile("" : "+s"(x_next));
            }
            if constexpr (CUR == 1 && m == turn_at(4)) set_scalar(w_read, w_next);
            if constexpr (CUR == 1 && m == turn_at(5)) {
                w_next = w_next == (kAhead - 1) * kWBytes ? 0u : w_next + kWBytes;
                asm volatile("" : "+s"(w_next));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // The ring keeps turning from tile to tile: the last kAhead steps of a tile load the first ones of the workgroup's next tile,
    // and the last half reads that tile's first fragments (not in the fused form, see below), so between two tiles only the
    // epilogue's instructions are exposed -- no workgroup start, no first trip to memory.
    auto k_step = [&](auto tail, auto read_next) __attribute__((always_inline)) {
        reserve_accumulators<4 * NI * NJ>();
        mfma_operands_ready();      // (fragments are copied where the loops meet)
        half(std::integral_constant<int, 0>{}, tail, std::true_type{});
        half(std::integral_constant<int, 1>{}, tail, read_next);
    };
    const std::integral_constant<int, -1> loading;
    const std::true_type reading;
    // In the fused form the first fragments of the next tile are read behind the epilogue instead, whose values need the
    // registers: 256 x 256 takes 236 vector registers so and the pair-by-pair rotation no scratch memory (256, and 108 bytes a
    // lane, with the fragments held through the epilogue: 96 x 96 tokens, 24 heads, pairs 33 + 31, the whole call 455 us for 439).
    constexpr bool kReadEarly = !is_fused(LAYOUT);
    const std::bool_constant<kReadEarly> reading_early;
    for (;;) {
        const uint32_t steps = n_k - kAhead;
        if (steps & 1u) k_step(loading, reading);
        uint32_t pairs = steps / 2u;      // two steps to a turn of the loop (a branch taken costs some 80 clocks)
        if (pairs > 0) {
#pragma unroll 1
            do {
                k_step(loading, reading);
                k_step(loading, reading);
            } while (--pairs > 0);
        }
        vt += walk.stride;
        const bool more = vt < walk.end;
        const TileCoord next = tile_at(a, more ? vt : walk.first);
        if (more) {
            load_from(next);
            uint32_t left = kAhead - 1;
#pragma unroll 1
            do k_step(loading, reading);
            while (--left > 0);
            k_step(loading, reading_early);
        } else {
            unrolled<kAhead>([&](auto s_c) __attribute__((always_inline)) {
                constexpr int follow = kAhead - 1 - decltype(s_c)::value;
                k_step(std::integral_constant<int, follow>{}, std::bool_constant<(follow > 0)>{});      // (the very last half reads nothing)
            });
        }
        mfma_results_ready();

        const GemmArgs& e = arguments_again();
        const uint32_t tok = tc.m0 + wave_t, feat = tc.f0 + wave_f;
        TileOut out;
        out.live_j = (int)min((uint32_t)NJ, tok < (uint32_t)e.M ? ((uint32_t)e.M - tok) / 16u : 0u);
        out.live_p = (int)min((uint32_t)NI / 2u, feat < (uint32_t)e.D ? ((uint32_t)e.D - feat) / 32u : 0u);
        if (out.live_p == 0) out.live_j = 0;
        out.n0 = (uint32_t)e.row_begin + tok;
        out.tl = lane & 15u;
        out.v8 = feat / 8u + (lane >> 4);
        uint16_t* y = e.y[tc.tensor];
        if constexpr (is_fused(LAYOUT)) {
            uint16_t* y2 = e.y2[tc.tensor];
            // the X slot of the step just finished is free until the next tile's first half loads into it again
            unsigned char* spare = smem + x_load;
            if (e.gamma[tc.tensor]) {     // the same for the whole workgroup: its barriers are taken by all or by none
                const uint16_t* gamma = e.gamma[tc.tensor];
                float* xch = reinterpret_cast<float*>(spare);
                if (e.d == 128u) store_normalised<NI, NJ, LAYOUT != OUT_FUSED_ANY, 128>(e, out, gamma, y, y2, xch, wave);
                else if (e.d == 64u) store_normalised<NI, NJ, LAYOUT != OUT_FUSED_ANY, 64>(e, out, gamma, y, y2, xch, wave);
                else if constexpr (NI == 8) store_normalised<NI, NJ, LAYOUT != OUT_FUSED_ANY, 256>(e, out, gamma, y, y2, xch, wave);
            } else if (e.sel_prev && tc.tensor == 0) {     // V (the first tensor of the launch), flagged on its way out
                const uint32_t mine = store_both<NI, NJ, true, LAYOUT == OUT_FUSED_STREAMED>(e, out, y, y2);
                // the verdicts of the two wavefronts that share the tokens
                uint32_t* verdicts = reinterpret_cast<uint32_t*>(spare);
                if (lane == 0) verdicts[wave] = mine;
                __syncthreads();
                const uint32_t any = verdicts[wave & ~1u] | verdicts[wave | 1u];
                if ((wave & 1u) == 0 && (int)lane < out.live_j)
                    e.sel_flag_bytes[(size_t)(out.n0 / 16u + lane) * 16u + tc.f0 / (uint32_t)TN] = (uint8_t)((any >> lane) & 1u);
                __syncthreads();     // before anybody loads into the slot again
            } else {
                store_both<NI, NJ, false, LAYOUT == OUT_FUSED_STREAMED>(e, out, y, y2);
            }
        } else {
            store_plain<NI, NJ, LAYOUT>(e, out, y);
        }
        if (!more) return;
        tc = next;
        if constexpr (!kReadEarly) {
#pragma unroll
            for (int r = 0; r < NREADS; ++r) read_frag(wf[0], xf[0], x_read, w_read, 0, r);
        }
    }
}

// Tile shapes (NI, NJ) that are built: 32 NI features x 32 NJ tokens.  The LONG ones lie between the others and are taken for
// launches of kLongSteps K steps and more only (plan_launch).
#define COCODIFF_PLAIN_TILES(F) F(8, 8) F(6, 9) F(6, 6) F(8, 4) F(4, 8) F(8, 3) F(4, 4) F(6, 3) F(4, 3) F(6, 2) F(4, 2) F(2, 2) F(2, 1)
#define COCODIFF_PLAIN_LONG_TILES(F) F(8, 6) F(6, 7) F(6, 5) F(6, 4) F(2, 3)
#define COCODIFF_FUSED_TILES(F) F(8, 8) F(8, 7) F(8, 6) F(8, 5) F(8, 4) F(8, 3) F(8, 2) F(4, 8) F(4, 4) F(4, 3) F(4, 2) F(4, 1)
#define COCODIFF_FUSED_LONG_TILES(F) F(4, 7) F(4, 6) F(4, 5)

// Host pointers of the kernels of one layout, in the order of the lists above; one source file each.
extern const void* const kSeqKernels[];
extern const void* const kChunkKernels[];
extern const void* const kHeadKernels[];
extern const void* const kFusedKernels[];
extern const void* const kFusedAnyKernels[];
extern const void* const kChunkStreamedKernels[];
extern const void* const kFusedStreamedKernels[];

}  // namespace cocodiff
