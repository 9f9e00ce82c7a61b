// The two Ulysses all-to-alls on one GPU (paper Section II-A): before attention, sequence-parallel ->
// head-parallel (pack the send chunks, unpack the received chunks head-major); after attention the way back
// (pack from the head-parallel tensor, unpack token-major).  Pure 128-bit permutation copies; HBM-bound.
//
// Units below are 16-byte vectors (8 bf16).  d8 = d/8 vectors per head row, D8 = D/8 per token row,
// row8 = Hp*d8 per chunk row, chunk8 = Ns*row8 per chunk.  A chunk always holds [Ns tokens][Hp heads][d] of
// one (token owner r, head owner p) pair; which of the two is the sender depends on the direction.
#include "internal.h"

namespace cocodiff {

constexpr int kThreads = 256;

struct PermuteArgs {
    uint32_t Ns, P, D8, d8, row8, chunk8, Hp;
    Divisor31 div_Ns, div_P, div_D8, div_d8, div_row8, div_chunk8, div_Hp, div_head8, div_ranks;
    uint32_t N;           // tokens in total
    uint32_t first;       // walk over x_seq: first token of the range; walk over x_hs: first head of the range
    uint32_t n_vec;       // vectors this launch moves
    int recv_major;
    uint32_t rank_begin, rank_count;     // the launch's ranks (buffer walks)
};

__device__ __forceinline__ uint32_t slot_of(uint32_t sender, uint32_t receiver, uint32_t P, int recv_major) {
    return recv_major ? receiver * P + sender : sender * P + receiver;
}

// Every kernel walks its OUTPUT linearly in 16-byte vectors: stores that run linearly through memory and loads that gather
// 512- or 256-byte pieces are faster than the other way round (cold, 57 MB tensors: 20 against 21.5 us).  Bound by HBM, and below
// some 20 MB by the launch and the start of its workgroups (an empty launch takes 2.6 us): so the index arithmetic is
// multiplications, and small tensors are moved with two vectors per lane (vectors_per_lane).
// A walk maps vector g of its output to where it is written (to) and where it is read (from).

// Exchange buffer -> sequence-parallel tensor [N][H][d] (second all-to-all: sender = head owner p, receiver = token
// owner r), linearly over the token range of the launch.
struct SeqFromBuf {
    static __device__ __forceinline__ void at(const PermuteArgs& a, uint32_t g, size_t& from, size_t& to) {
        const uint32_t tl = div_by(g, a.div_D8);      // token within the range
        const uint32_t v = g - tl * a.D8;             // vector within the token row
        const uint32_t n = a.first + tl;              // global token
        const uint32_t r = div_by(n, a.div_Ns);       // token owner
        const uint32_t m = n - r * a.Ns;              // token within the rank
        const uint32_t p = div_by(v, a.div_row8);     // head owner
        const uint32_t c = v - p * a.row8;            // (hl, i) within the chunk row
        to = (size_t)n * a.D8 + v;
        from = (size_t)slot_of(p, r, a.P, a.recv_major) * a.chunk8 + m * a.row8 + c;
    }
};

// Exchange buffer -> head-parallel tensor [H][N][d] (first all-to-all: sender = token owner r, receiver = head owner
// p), linearly over the head range of the launch.
struct HeadsFromBuf {
    static __device__ __forceinline__ void at(const PermuteArgs& a, uint32_t g, size_t& from, size_t& to) {
        const uint32_t head8 = a.N * a.d8;            // vectors per head slab
        const uint32_t hl_range = div_by(g, a.div_head8);
        const uint32_t rem = g - hl_range * head8;
        const uint32_t h = a.first + hl_range;        // global head
        const uint32_t n = div_by(rem, a.div_d8);     // global token
        const uint32_t i8 = rem - n * a.d8;
        const uint32_t p = div_by(h, a.div_Hp);       // head owner
        const uint32_t hl = h - p * a.Hp;
        const uint32_t r = div_by(n, a.div_Ns);       // token owner
        const uint32_t m = n - r * a.Ns;
        to = (size_t)a.first * head8 + g;
        from = (size_t)slot_of(r, p, a.P, a.recv_major) * a.chunk8 + m * a.row8 + hl * a.d8 + i8;
    }
};

// The packing directions: vector g of the launch is vector g of the chunks the launch's ranks send, in buffer order.
// Sequence-parallel tensor -> exchange buffer (first all-to-all): the senders are the token owners r of the rank range.
struct BufFromSeq {
    static __device__ __forceinline__ void at(const PermuteArgs& a, uint32_t g, size_t& from, size_t& to) {
        const uint32_t ch = div_by(g, a.div_chunk8), rem = g - ch * a.chunk8;       // chunk of the launch, vector inside it
        // send-major: chunks (r, p) with p fastest; receive-major: (p, r) with r fastest
        const uint32_t q = a.recv_major ? div_by(ch, a.div_ranks) : div_by(ch, a.div_P);
        const uint32_t r = a.rank_begin + (a.recv_major ? ch - q * a.rank_count : q);
        const uint32_t p = a.recv_major ? q : ch - q * a.P;
        const uint32_t m = div_by(rem, a.div_row8), c = rem - m * a.row8;
        from = (size_t)(r * a.Ns + m) * a.D8 + p * a.row8 + c;
        to = (size_t)slot_of(r, p, a.P, a.recv_major) * a.chunk8 + rem;
    }
};

// Head-parallel tensor -> exchange buffer (second all-to-all): the senders are the head owners p of the rank range.
struct BufFromHeads {
    static __device__ __forceinline__ void at(const PermuteArgs& a, uint32_t g, size_t& from, size_t& to) {
        const uint32_t ch = div_by(g, a.div_chunk8), rem = g - ch * a.chunk8;
        // send-major: chunks (p, r) with r fastest; receive-major: (r, p) with p fastest
        const uint32_t q = a.recv_major ? div_by(ch, a.div_ranks) : div_by(ch, a.div_P);
        const uint32_t p = a.rank_begin + (a.recv_major ? ch - q * a.rank_count : q);
        const uint32_t r = a.recv_major ? q : ch - q * a.P;
        const uint32_t m = div_by(rem, a.div_row8), c = rem - m * a.row8;           // token within the rank; (hl, i) within the chunk row
        const uint32_t hl = div_by(c, a.div_d8), i8 = c - hl * a.d8;
        from = ((size_t)(p * a.Hp + hl) * a.N + r * a.Ns + m) * a.d8 + i8;
        to = (size_t)slot_of(p, r, a.P, a.recv_major) * a.chunk8 + rem;
    }
};

template <typename Walk, int U, bool NT_LD, bool NT_ST>
__global__ void __launch_bounds__(kThreads) permute_kernel(const vec16* __restrict__ in, vec16* __restrict__ out, PermuteArgs a) {
    const uint32_t g0 = blockIdx.x * (kThreads * U) + threadIdx.x;
    vec16 v[U];
    size_t to[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint32_t g = g0 + k * kThreads;
        if (g < a.n_vec) {
            size_t from;
            Walk::at(a, g, from, to[k]);
            v[k] = ld_vec<NT_LD>(in + from);
        }
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
        if (g0 + k * kThreads < a.n_vec) st_vec<NT_ST>(out + to[k], v[k]);
}

// Two vectors per lane below 20 MB.  A plain copy, cold, one and two per lane: 4.7 MB 3.0 and 3.1 us, 11.3 MB 5.5 and 5.0, 14.2 MB 6.4
// and 5.4, 28.3 MB 11.1 and 11.2, 56.6 MB 19.8 and 20.1, 127 MB 41.8 and 43.2; four are slower at every size.
static int vectors_per_lane(uint32_t n_vec) { return n_vec < (20u << 20) / 16u ? 2 : 1; }

static int check_permute(const cocodiff_shape* s, const void* in, const void* out, int slot_order, const char* who) {
    int rc = check_shape(s);
    if (rc != COCODIFF_OK) return rc;
    if (!in || !out) return fail(COCODIFF_ERR_NULL, "%s: NULL tensor pointer", who);
    if (!aligned16(in) || !aligned16(out)) return fail(COCODIFF_ERR_ALIGN, "%s: pointers must be 16-byte aligned", who);
    if (slot_order != COCODIFF_SEND_MAJOR && slot_order != COCODIFF_RECV_MAJOR)
        return fail(COCODIFF_ERR_SHAPE, "%s: slot_order (%d) must be SEND_MAJOR or RECV_MAJOR", who, slot_order);
    if ((int64_t)s->N * s->D / 8 >= (int64_t)1 << 31)
        return fail(COCODIFF_ERR_SHAPE, "%s: N*D/8 must be below 2^31", who);
    return COCODIFF_OK;
}

static PermuteArgs make_args(const cocodiff_shape* s, int slot_order) {
    PermuteArgs a;
    a.Ns = s->N / s->P;
    a.P = s->P;
    a.D8 = s->D / 8;
    a.d8 = s->d / 8;
    a.Hp = s->H / s->P;
    a.row8 = a.Hp * a.d8;
    a.chunk8 = a.Ns * a.row8;
    a.N = s->N;
    a.first = 0;
    a.n_vec = 0;
    a.recv_major = slot_order == COCODIFF_RECV_MAJOR;
    a.rank_begin = (uint32_t)s->rank_begin;
    a.rank_count = (uint32_t)s->rank_count;
    // (every dividend is below N * D / 8, which is below 2^31)
    a.div_Ns = make_divisor31(a.Ns);
    a.div_P = make_divisor31(a.P);
    a.div_D8 = make_divisor31(a.D8);
    a.div_d8 = make_divisor31(a.d8);
    a.div_row8 = make_divisor31(a.row8);
    a.div_chunk8 = make_divisor31(a.chunk8);
    a.div_Hp = make_divisor31(a.Hp);
    a.div_head8 = make_divisor31(a.N * a.d8);
    a.div_ranks = make_divisor31(a.rank_count);
    return a;
}

template <typename Walk>
static int launch_permute(const PermuteArgs& a, const void* in, void* out, void* stream, const char* who) {
    const size_t touched = (size_t)a.n_vec * 32;
    with_policy(stream_loads(touched), stream_stores(touched), [&](auto L, auto S) {
        auto launch = [&](auto u_c) {
            constexpr int U = decltype(u_c)::value;
            const dim3 grid((a.n_vec + kThreads * U - 1) / (kThreads * U));
            hipLaunchKernelGGL((permute_kernel<Walk, U, decltype(L)::value, decltype(S)::value>), grid, dim3(kThreads), 0, as_stream(stream),
                               (const vec16*)in, (vec16*)out, a);
        };
        if (vectors_per_lane(a.n_vec) == 2) launch(std::integral_constant<int, 2>{});
        else launch(std::integral_constant<int, 1>{});
    });
    return check_launch(who);
}

// Between the sequence-parallel tensor and the buffer; the ranks of the shape's range are token owners.
template <typename Walk>
static int launch_seq_side(const cocodiff_shape* shape, const void* in, void* out, int slot_order, void* stream, const char* who) {
    int rc = check_permute(shape, in, out, slot_order, who);
    if (rc != COCODIFF_OK) return rc;
    PermuteArgs a = make_args(shape, slot_order);
    a.first = shape->rank_begin * a.Ns;
    a.n_vec = (uint32_t)shape->rank_count * a.Ns * a.D8;
    return launch_permute<Walk>(a, in, out, stream, who);
}

// Between the head-parallel tensor and the buffer; the ranks of the shape's range are head owners.
template <typename Walk>
static int launch_head_side(const cocodiff_shape* shape, const void* in, void* out, int slot_order, void* stream, const char* who) {
    int rc = check_permute(shape, in, out, slot_order, who);
    if (rc != COCODIFF_OK) return rc;
    PermuteArgs a = make_args(shape, slot_order);
    a.first = shape->rank_begin * a.Hp;
    a.n_vec = (uint32_t)shape->rank_count * a.Hp * a.N * a.d8;
    return launch_permute<Walk>(a, in, out, stream, who);
}

}  // namespace cocodiff

using namespace cocodiff;

extern "C" int cocodiff_a2a_pack(const cocodiff_shape* shape, const cocodiff_bf16* x_seq, cocodiff_bf16* xbuf,
                                 int slot_order, void* stream) {
    return launch_seq_side<BufFromSeq>(shape, x_seq, xbuf, slot_order, stream, "a2a_pack");
}

extern "C" int cocodiff_a2a_unpack(const cocodiff_shape* shape, const cocodiff_bf16* xbuf, cocodiff_bf16* x_hs,
                                   int slot_order, void* stream) {
    return launch_head_side<HeadsFromBuf>(shape, xbuf, x_hs, slot_order, stream, "a2a_unpack");
}

extern "C" int cocodiff_a2a_pack_hs(const cocodiff_shape* shape, const cocodiff_bf16* y_hs, cocodiff_bf16* xbuf,
                                    int slot_order, void* stream) {
    return launch_head_side<BufFromHeads>(shape, y_hs, xbuf, slot_order, stream, "a2a_pack_hs");
}

extern "C" int cocodiff_a2a_unpack_seq(const cocodiff_shape* shape, const cocodiff_bf16* xbuf, cocodiff_bf16* y_seq,
                                       int slot_order, void* stream) {
    return launch_seq_side<SeqFromBuf>(shape, xbuf, y_seq, slot_order, stream, "a2a_unpack_seq");
}
