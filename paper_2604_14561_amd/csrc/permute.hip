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

// Every kernel walks its OUTPUT linearly in 16-byte vectors: stores that run linearly through memory and loads that gather
// 512- or 256-byte pieces are faster than the other way round (cold, 57 MB tensors: 20 against 21.5 us).  Bound by HBM, and below
// some 20 MB by the launch and the start of its workgroups (an empty launch takes 2.6 us).
// A launch's arguments are not on chip when it starts, whoever reads a line of them first waits for memory; so they are few
// (the chunk strides folded into two factors), and all are asked for before the first branch (settled).  Twice as many, read where
// they were needed, cost a call 0.3 to 0.6 us: the stand-alone calls at 4608 x 2048 189.2 -> 186.8 us, a small pack and unpack pair
// 11.0 -> 9.8.
//
// A walk maps vector g of its output to where it is read (from) and written (to): all below N*D/8 < 2^31, in arithmetic modulo 2^32.
// rs, ps: what one token owner r, one head owner p further means in the buffer, in vectors.

// Exchange buffer -> sequence-parallel tensor [N][H][d] (second all-to-all: sender = head owner p, receiver = token
// owner r), linearly over the token range of the launch.
struct SeqFromBuf {
    uint32_t n_vec, D8, first, to0, row8;       // first: first token of the range
    uint32_t per_r, per_p;                      // rs - chunk8, ps - row8: the rest of them is in n * row8 and v
    Divisor31 div_D8, div_Ns, div_row8;
    __device__ __forceinline__ void at(uint32_t g, uint32_t& from, uint32_t& to) const {
        const uint32_t tl = div_by(g, div_D8), v = g - tl * D8;       // token within the range, vector within the token row
        const uint32_t n = first + tl, r = div_by(n, div_Ns), p = div_by(v, div_row8);
        from = n * row8 + r * per_r + v + p * per_p;
        to = to0 + g;
    }
};

// Exchange buffer -> head-parallel tensor [H][N][d] (first all-to-all: sender = token owner r, receiver = head owner
// p), linearly over the head range of the launch.
struct HeadsFromBuf {
    uint32_t n_vec, head8, first, to0, row8, d8;       // head8: vectors per head slab; first: first head of the range
    uint32_t per_r, per_p;                             // as above, of n * row8 and h * d8
    Divisor31 div_head8, div_d8, div_Ns, div_Hp;
    __device__ __forceinline__ void at(uint32_t g, uint32_t& from, uint32_t& to) const {
        const uint32_t hl_range = div_by(g, div_head8), rem = g - hl_range * head8, h = first + hl_range;
        const uint32_t n = div_by(rem, div_d8), i8 = rem - n * d8, r = div_by(n, div_Ns), p = div_by(h, div_Hp);
        from = n * row8 + r * per_r + h * d8 + p * per_p + i8;
        to = to0 + g;
    }
};

// The packing directions: vector g of the launch is vector g of the chunks the launch's ranks send, in buffer order: chunk (hi, lo)
// with lo fastest, one of the two the sender within the rank range, the other the receiver.
struct Chunks {
    uint32_t n_vec, chunk8, row8, n_lo;
    uint32_t from_hi, from_lo, from0;           // where chunk (hi, lo) begins in the tensor
    uint32_t to_hi, to0;                        // and in the buffer, where lo steps by chunk8
    Divisor31 div_chunk8, div_lo, div_row8;
    __device__ __forceinline__ void split(uint32_t g, uint32_t& from, uint32_t& to, uint32_t& m, uint32_t& c) const {
        const uint32_t ch = div_by(g, div_chunk8), rem = g - ch * chunk8, hi = div_by(ch, div_lo), lo = ch - hi * n_lo;
        m = div_by(rem, div_row8);              // token within the rank
        c = rem - m * row8;                     // (hl, i) within the chunk row
        from = from0 + hi * from_hi + lo * from_lo;
        to = to0 + hi * to_hi + lo * chunk8 + rem;
    }
};

// Sequence-parallel tensor -> exchange buffer (first all-to-all): the senders are the token owners r of the rank range.
struct BufFromSeq : Chunks {
    uint32_t D8;
    __device__ __forceinline__ void at(uint32_t g, uint32_t& from, uint32_t& to) const {
        uint32_t m, c;
        split(g, from, to, m, c);
        from += m * D8 + c;
    }
};

// Head-parallel tensor -> exchange buffer (second all-to-all): the senders are the head owners p of the rank range.
struct BufFromHeads : Chunks {
    uint32_t d8, per_head;                      // per_head: vectors per head slab, less the d8 that c counts
    Divisor31 div_d8;
    __device__ __forceinline__ void at(uint32_t g, uint32_t& from, uint32_t& to) const {
        uint32_t m, c;
        split(g, from, to, m, c);
        from += m * d8 + c + div_by(c, div_d8) * per_head;
    }
};

// The values are there before anything after this is decided: what they are formed from cannot be moved behind a branch.
__device__ __forceinline__ void settled(uint32_t& a, uint32_t& b) { asm volatile("" : "+v"(a), "+v"(b)); }

template <typename Walk, int U, bool NT_LD, bool NT_ST>
__global__ void __launch_bounds__(kThreads) permute_kernel(const vec16* __restrict__ in, vec16* __restrict__ out, Walk a) {
    const uint32_t g0 = blockIdx.x * (kThreads * U) + threadIdx.x;
    vec16 v[U];
    uint32_t from[U], to[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        a.at(min(g0 + k * kThreads, a.n_vec - 1u), from[k], to[k]);
        settled(from[k], to[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
        if (g0 + k * kThreads < a.n_vec) v[k] = ld_vec<NT_LD>(in + from[k]);
#pragma unroll
    for (int k = 0; k < U; ++k)
        if (g0 + k * kThreads < a.n_vec) st_vec<NT_ST>(out + to[k], v[k]);
}

// Two vectors per lane where all lanes that the chip holds (256 units x 2048) move the launch at two each but not at one: 8 to 16 MiB
// of output.  There the launch is one residency of the chip instead of two; below, one vector per lane is one residency already, and
// above, neither is.  Cold, from a graph, three geometries (24 heads of 128 on 12 ranks, 18 of 64 on 9, 16 of 128 on one), two vectors
// against one, mean and range over sizes:
//   4 to 8 MiB      pack and the unpack that reads its buffer -1.4 % (-6 .. +4)     a walk alone +0.8 % (-5 .. +4)
//   8 to 12 MiB                                               -7.2 % (-14 .. -1)                 -4.5 % (-11 .. 0)
//   12 to 16 MiB                                              -3.6 % (-8 .. +1)                  -3.2 % (-12 .. +4)
//   16 to 24 MiB                                              +3.7 % (+1 .. +6)                  -0.4 % (-7 .. +7)
// (pack and unpack of 12 MiB 13.0 -> 11.8 us, of 18 MiB 17.4 -> 18.2.)  Four are slower at every size.
constexpr uint32_t kResidentLanes = 256u * 2048u;
static int vectors_per_lane(uint32_t n_vec) { return n_vec >= kResidentLanes && n_vec < 2u * kResidentLanes ? 2 : 1; }

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

// Sizes in vectors, and the buffer's strides: slot (receiver, sender) or (sender, receiver), the second fastest.
struct Sizes {
    uint32_t Ns, D8, d8, Hp, row8, chunk8, head8, begin, count, rs, ps;
    Sizes(const cocodiff_shape* s, int slot_order, bool r_sends) {
        Ns = (uint32_t)(s->N / s->P);
        D8 = (uint32_t)s->D / 8u;
        d8 = (uint32_t)s->d / 8u;
        Hp = (uint32_t)(s->H / s->P);
        row8 = Hp * d8;
        chunk8 = Ns * row8;
        head8 = (uint32_t)s->N * d8;
        begin = (uint32_t)s->rank_begin;
        count = (uint32_t)s->rank_count;
        const bool r_fastest = (slot_order == COCODIFF_RECV_MAJOR) == r_sends;
        rs = r_fastest ? chunk8 : (uint32_t)s->P * chunk8;
        ps = r_fastest ? (uint32_t)s->P * chunk8 : chunk8;
    }
};

template <typename Walk>
static int launch_permute(const Walk& a, const void* in, void* out, void* stream, const char* who) {
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

// The chunks that `z.count` senders from z.begin on send to P receivers each, in buffer order.  sender, receiver: what one sender and
// one receiver further means in the tensor; sender_buf: and one sender further in the buffer.
static void set_chunks(Chunks* a, const Sizes& z, uint32_t P, bool recv_major, uint32_t sender, uint32_t receiver, uint32_t sender_buf) {
    a->n_vec = z.count * P * z.chunk8;
    a->chunk8 = z.chunk8;
    a->row8 = z.row8;
    a->n_lo = recv_major ? z.count : P;
    a->from_hi = recv_major ? receiver : sender;
    a->from_lo = recv_major ? sender : receiver;
    a->from0 = z.begin * sender;
    a->to_hi = P * z.chunk8;
    a->to0 = z.begin * sender_buf;
    // (every dividend is below N * D / 8, which is below 2^31)
    a->div_chunk8 = make_divisor31(z.chunk8);
    a->div_lo = make_divisor31(a->n_lo);
    a->div_row8 = make_divisor31(z.row8);
}

}  // namespace cocodiff

using namespace cocodiff;

extern "C" int cocodiff_a2a_pack(const cocodiff_shape* shape, const cocodiff_bf16* x_seq, cocodiff_bf16* xbuf,
                                 int slot_order, void* stream) {
    const int rc = check_permute(shape, x_seq, xbuf, slot_order, "a2a_pack");
    if (rc != COCODIFF_OK) return rc;
    const Sizes z(shape, slot_order, true);
    BufFromSeq a;
    set_chunks(&a, z, (uint32_t)shape->P, slot_order == COCODIFF_RECV_MAJOR, z.Ns * z.D8, z.row8, z.rs);
    a.D8 = z.D8;
    return launch_permute(a, x_seq, xbuf, stream, "a2a_pack");
}

extern "C" int cocodiff_a2a_unpack(const cocodiff_shape* shape, const cocodiff_bf16* xbuf, cocodiff_bf16* x_hs,
                                   int slot_order, void* stream) {
    const int rc = check_permute(shape, xbuf, x_hs, slot_order, "a2a_unpack");
    if (rc != COCODIFF_OK) return rc;
    const Sizes z(shape, slot_order, true);
    HeadsFromBuf a;
    a.n_vec = z.count * z.Hp * z.head8;
    a.head8 = z.head8;
    a.first = z.begin * z.Hp;
    a.to0 = a.first * z.head8;
    a.row8 = z.row8;
    a.d8 = z.d8;
    a.per_r = z.rs - z.chunk8;
    a.per_p = z.ps - z.row8;
    a.div_head8 = make_divisor31(z.head8);
    a.div_d8 = make_divisor31(z.d8);
    a.div_Ns = make_divisor31(z.Ns);
    a.div_Hp = make_divisor31(z.Hp);
    return launch_permute(a, xbuf, x_hs, stream, "a2a_unpack");
}

extern "C" int cocodiff_a2a_pack_hs(const cocodiff_shape* shape, const cocodiff_bf16* y_hs, cocodiff_bf16* xbuf,
                                    int slot_order, void* stream) {
    const int rc = check_permute(shape, y_hs, xbuf, slot_order, "a2a_pack_hs");
    if (rc != COCODIFF_OK) return rc;
    const Sizes z(shape, slot_order, false);
    BufFromHeads a;
    set_chunks(&a, z, (uint32_t)shape->P, slot_order == COCODIFF_RECV_MAJOR, z.Hp * z.head8, z.Ns * z.d8, z.ps);
    a.d8 = z.d8;
    a.per_head = z.head8 - z.d8;
    a.div_d8 = make_divisor31(z.d8);
    return launch_permute(a, y_hs, xbuf, stream, "a2a_pack_hs");
}

extern "C" int cocodiff_a2a_unpack_seq(const cocodiff_shape* shape, const cocodiff_bf16* xbuf, cocodiff_bf16* y_seq,
                                       int slot_order, void* stream) {
    const int rc = check_permute(shape, xbuf, y_seq, slot_order, "a2a_unpack_seq");
    if (rc != COCODIFF_OK) return rc;
    const Sizes z(shape, slot_order, false);
    SeqFromBuf a;
    a.n_vec = z.count * z.Ns * z.D8;
    a.D8 = z.D8;
    a.first = z.begin * z.Ns;
    a.to0 = a.first * z.D8;
    a.row8 = z.row8;
    a.per_r = z.rs - z.chunk8;
    a.per_p = z.ps - z.row8;
    a.div_D8 = make_divisor31(z.D8);
    a.div_Ns = make_divisor31(z.Ns);
    a.div_row8 = make_divisor31(z.row8);
    return launch_permute(a, xbuf, y_seq, stream, "a2a_unpack_seq");
}
