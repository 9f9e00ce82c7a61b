"""Performance cases: what a program that uses this package has it do, through the public entry points.

A case is a dict of plain values: `kind` names one of the call sequences below, the rest gives its sizes (`grid` is the
token grid, last axis fastest, N = its product; H heads of d; P logical ranks).  The sequences are those of one
attention layer in one denoising step:

  layer   everything in one call, as a single GPU that holds all ranks runs it: Q, K, V projected, Q and K normalised and
          rotated, every tensor in its exchange buffer and head-parallel, V's changed tiles selected and gathered
  vfirst  the V-First order with the exchange between sender and receiver: V packed first, then Q and K; the receiver
          unpacks V with the selection inside and Q and K with the normalisation inside
  calls   the stand-alone calls one after the other, a program that composes the steps itself
  rank    one rank's own share, what each process of a one-process-per-GPU job calls: its token rows projected into its
          send chunks, its heads unpacked from its receive chunks, its slab of V selected
  vmajor  the V-Major update of the cached tensors by 16-token tiles: selection on V, Q and K gathered by V's list, all
          three scattered into the caches
  tokens  the same update by single tokens: distance per token, the largest kept (as many as the cache schedule says for
          the denoising step), gather and scatter by that list
  back    the second all-to-all after attention: pack the head-parallel result, unpack it token-major
"""
import math

import torch

import paper_2604_14561_amd as cd

TILE = 16           # tokens per selection tile
EPS = 1e-6
THETA = 10000.0
# Selection threshold.  Between two steps every token drifts a little (sigma 0.002 on the hidden state, values of V move by
# less than 0.06 with their rounding to bf16) and the changed ones move by sigma 0.5: the threshold lies between.
TAU = 0.1
DRIFT, CHANGE = 0.002, 0.5
N_STEPS, WARMUP_STEPS, SYNC_EVERY = 50, 5, 10      # the denoising run of the cache schedule


def listed():
    return [
        # the smallest layer of the configurations: latency of the call and its launches
        dict(name="layer tiny", kind="layer", grid="16x16", H=4, d=64, P=2, changed=0.25),
        # image layers, 24 heads of 128, 12 ranks: 768 x 768 and 1536 x 1536 pixels (16 pixels a token and axis)
        dict(name="layer 768", kind="layer", grid="48x48", H=24, d=128, P=12, changed=0.30),
        dict(name="layer 1536", kind="layer", grid="96x96", H=24, d=128, P=12, changed=0.20),
        # a 1280 x 720 image and heads of 64: no size is a multiple of the projection's tiles
        dict(name="layer 720p", kind="layer", grid="45x80", H=18, d=64, P=9, changed=0.20),
        # a video latent, three rotary axes: the largest workload
        dict(name="layer video", kind="layer", grid="16x60x104", H=24, d=128, P=24, changed=0.15),
        # 2304 x 2304 pixels with the exchange between sender and receiver
        dict(name="vfirst 2304", kind="vfirst", grid="144x144", H=24, d=128, P=12, changed=0.10),
        # the steps called one by one on a 768 x 768 image
        dict(name="calls 768", kind="calls", grid="48x48", H=24, d=128, P=12, changed=0.30),
        # one of 12 ranks at 1536 x 1536 (768 tokens), one of 8 on the video latent (12480 tokens)
        dict(name="rank 1536", kind="rank", grid="96x96", H=24, d=128, P=12, changed=0.20),
        dict(name="rank video", kind="rank", grid="16x60x104", H=24, d=128, P=8, changed=0.15),
        # cache updates: by tiles on a whole 1536 x 1536 image, by tokens on one of 8 ranks of the video latent
        dict(name="vmajor 1536", kind="vmajor", grid="96x96", H=24, d=128, P=12, changed=0.20),
        dict(name="tokens video", kind="tokens", grid="16x60x104", H=24, d=128, P=8, step=27),
        # the way back after attention at 2304 x 2304
        dict(name="back 2304", kind="back", grid="144x144", H=24, d=128, P=12),
    ]


def draw(rng):
    """A case of the same ranges: 256 to about 80000 tokens, 256 to 3072 features, heads of 64 and 128, any rank count that
    divides the heads, two- and three-axis grids."""
    kind = rng.choice(("layer", "layer", "layer", "vfirst", "calls", "rank", "rank", "vmajor", "tokens", "back"))
    d = rng.choice((64, 128, 128))
    if kind == "calls":      # whole wavefronts of 16-byte vectors per token row
        H = rng.randint(1, 6) * (512 // d)
    else:
        H = rng.randint(256 // d, 3072 // d)
    P = rng.choice([p for p in range(1, min(H, 24) + 1) if H % p == 0])
    # a grid of about as many tokens as wanted whose ranks hold whole selection tiles: the best of 32 first sides
    want = math.exp(rng.uniform(math.log(256), math.log(60000 if kind == "calls" else 80000)))
    frames = rng.randint(2, 24) if want > 2000 and rng.random() < 0.3 else 1
    grids = []
    for _ in range(32):
        h = max(2, round(math.sqrt(want / frames) * math.exp(rng.uniform(-0.4, 0.4))))
        step = 16 * P // math.gcd(16 * P, frames * h)
        w = max(1, round(want / (frames * h * step))) * step
        grids.append(([frames] if frames > 1 else []) + [h, w])
    grid = min(grids, key=lambda g: abs(math.log(math.prod(g) / want)))
    case = dict(kind=kind, grid="x".join(str(a) for a in grid), H=H, d=d, P=P)
    if kind == "tokens":
        case["step"] = rng.choice([s for s in range(WARMUP_STEPS + 1, N_STEPS) if s % SYNC_EVERY])
    elif kind != "back":
        case["changed"] = round(rng.uniform(0.05, 0.35), 2)
    return case


def _sizes(case):
    grid = [int(a) for a in case["grid"].split("x")]
    return grid, math.prod(grid), case["H"], case["d"], case["P"]


def _changed_tiles(case):
    return round(case["changed"] * (_sizes(case)[1] // TILE))


def _kept_tokens(case):
    _, N, _, _, P = _sizes(case)
    return cd.cache_active_count(case["step"], N_STEPS, WARMUP_STEPS, SYNC_EVERY, N // P)


class _Inputs:
    """Seeded device inputs: values as the path meets them (hidden states N(0, 1), weights N(0, 1/D), gains near 1)."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape, scale=1.0, shift=0.0):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.bfloat16).mul_(scale).add_(shift)

    def one_step_before(self, x, axis, unit, count):
        """`x` as it was a step earlier: a small drift everywhere, a real change in `count` units of `unit` rows of `axis`."""
        rows = x.shape[axis]
        sigma = torch.full((rows // unit,), DRIFT, device="cuda", dtype=torch.bfloat16)
        sigma[torch.randperm(rows // unit, generator=self.gen, device="cuda")[:count]] = CHANGE
        shape = [1] * x.dim()
        shape[axis] = rows
        return x + self.normal(*x.shape) * sigma.repeat_interleave(unit).view(shape)


def _new(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, device="cuda", dtype=dtype)


class _State:
    pass


def _selection_outputs(s, S, N, W, cap):
    s.flags, s.idx, s.n_active = (_new(n, dtype=torch.int32) for n in (N // TILE, N // TILE, 1))
    s.compact, s.cap = _new(S, cap * TILE, W), cap


def prepare(case, seed):
    grid, N, H, d, P = _sizes(case)
    D, kind = H * d, case["kind"]
    make, s = _Inputs(seed), _State()
    s.run, s.N, s.H, s.d, s.P = _RUN[kind], N, H, d, P
    s.shape = cd.Shape.make(N, D, H, d, P)
    if kind == "back":
        s.y_hs, s.buf, s.y_seq = make.normal(H, N, d), _new(N * D), _new(N, H, d)
        return s
    if kind == "vmajor":
        s.v = make.normal(H, N, d)
        s.v_prev = make.one_step_before(s.v, 1, TILE, _changed_tiles(case))
        s.q, s.k = make.normal(H, N, d), make.normal(H, N, d)
        s.caches = [make.normal(H, N, d), make.normal(H, N, d), s.v_prev.clone()]
        _selection_outputs(s, H, N, d, N // TILE)
        s.q_compact, s.k_compact = torch.zeros_like(s.compact), torch.zeros_like(s.compact)
        s.ws = _new(max(16, cd.vmajor_select_workspace_bytes(H, N, d, TILE)), dtype=torch.uint8)
        return s
    if kind == "tokens":
        s.Ns, s.keep, s.D = N // P, _kept_tokens(case), D
        s.v = make.normal(s.Ns, D)
        s.v_prev = make.one_step_before(s.v, 0, 1, s.keep)
        s.q, s.k = make.normal(s.Ns, D), make.normal(s.Ns, D)
        s.caches = [make.normal(s.Ns, D), make.normal(s.Ns, D), s.v_prev.clone()]
        s.compact = [_new(s.keep, D) for _ in range(3)]
        s.metric = _new(s.Ns, dtype=torch.float32)
        s.idx, s.n_active = _new(s.Ns, dtype=torch.int32), _new(1, dtype=torch.int32)
        return s

    # the sequences that project
    s.x = make.normal(N, D)
    s.wq, s.wk, s.wv = (make.normal(D, D, scale=D ** -0.5) for _ in range(3))
    s.gq, s.gk = make.normal(d, scale=0.1, shift=1.0), make.normal(d, scale=0.1, shift=1.0)
    pairs = [d // 4, d // 4] if len(grid) == 2 else [d // 8, 3 * d // 16, 3 * d // 16]
    s.table = torch.from_numpy(cd.rope_table(grid, pairs, THETA)).cuda()
    s.rope = cd.Rope.make(grid, pairs, THETA, s.table.data_ptr())
    s.bufs = [_new(N * D) for _ in range(3)]           # exchange buffers and head-parallel tensors of Q, K, V
    s.hs = [_new(H, N, d) for _ in range(3)]
    if kind == "rank":
        r, Hp = P // 2, H // P
        s.mine = cd.Shape.make(N, D, H, d, P, rank_begin=r, rank_count=1)
        s.received = [_new(P * P, N // P, Hp, d) for _ in range(3)]        # RECV_MAJOR: this rank's chunks are slots r*P ...
        for t in s.received:
            t[r * P:(r + 1) * P] = make.normal(P, N // P, Hp, d)
        v = s.received[2][r * P:(r + 1) * P].reshape(N, Hp, d).transpose(0, 1).contiguous()
        s.v_prev = make.one_step_before(v, 1, TILE, _changed_tiles(case))
        s.sent = [b.view(P, -1)[r] for b in s.bufs]
        s.own = [t[r * Hp:(r + 1) * Hp] for t in s.hs]
        s.Hp = Hp
        _selection_outputs(s, Hp, N, d, N // TILE)
        s.ws = _new(max(16, cd.vmajor_select_workspace_bytes(Hp, N, d, TILE)), dtype=torch.uint8)
        return s
    x_prev = make.one_step_before(s.x, 0, TILE, _changed_tiles(case))
    s.v_prev = torch.mm(x_prev, s.wv.t()).view(N, H, d).transpose(0, 1).contiguous()
    if kind == "calls":
        s.qkv = [_new(N, D) for _ in range(3)]
    _selection_outputs(s, H, N, d, N // TILE)
    s.ws = _new(max(16, cd.vmajor_select_workspace_bytes(H, N, d, TILE), cd.qkv_proj_fused_select_workspace_bytes(s.shape, TILE)),
                dtype=torch.uint8)
    return s


def _layer(s):
    cd.qkv_proj_fused_select(s.shape, s.x, s.wq, s.wk, s.wv, s.gq, s.gk, EPS, s.rope, s.bufs[0], s.bufs[1], s.bufs[2], cd.RECV_MAJOR,
                             s.hs[0], s.hs[1], s.hs[2], s.v_prev, TILE, TAU, s.flags, s.idx, s.n_active, s.compact, s.cap, s.ws)
    return s.bufs, s.hs, s.flags, s.idx, s.n_active, s.compact


def _vfirst(s):
    cd.qkv_proj_pack(s.shape, s.x, None, None, s.wv, None, None, s.bufs[2], cd.RECV_MAJOR)
    cd.qkv_proj_pack(s.shape, s.x, s.wq, s.wk, None, s.bufs[0], s.bufs[1], None, cd.RECV_MAJOR)
    cd.a2a_unpack_select(s.shape, s.bufs[2], cd.RECV_MAJOR, s.hs[2], s.v_prev, TILE, TAU, s.flags, s.idx, s.n_active, s.compact, s.cap,
                         s.ws)
    cd.a2a_unpack_norm_rope(s.shape, s.bufs[0], s.bufs[1], s.hs[0], s.hs[1], s.gq, s.gk, EPS, s.rope, cd.RECV_MAJOR)
    return s.bufs, s.hs, s.flags, s.idx, s.n_active, s.compact


def _calls(s):
    q, k, v = s.qkv
    cd.qkv_proj(s.shape, s.x, None, None, s.wv, None, None, v)
    cd.qkv_proj(s.shape, s.x, s.wq, s.wk, None, q, k, None)
    cd.qk_norm_rope(s.shape, q, k, s.gq, s.gk, EPS, s.rope)
    for t, buf, hs in zip((v, q, k), (s.bufs[2], s.bufs[0], s.bufs[1]), (s.hs[2], s.hs[0], s.hs[1])):
        cd.a2a_pack(s.shape, t, buf, cd.SEND_MAJOR)
        cd.a2a_unpack(s.shape, buf, hs, cd.SEND_MAJOR)
    cd.vmajor_select(s.H, s.N, s.d, TILE, s.hs[2], s.v_prev, TAU, s.flags, s.idx, s.n_active, s.compact, s.cap, s.ws)
    return s.qkv, s.bufs, s.hs, s.flags, s.idx, s.n_active, s.compact


def _rank(s):
    # sender: V's chunks first, then Q's and K's, normalised
    cd.qkv_proj_pack(s.mine, s.x, None, None, s.wv, None, None, s.bufs[2], cd.SEND_MAJOR)
    cd.qkv_proj_fused(s.mine, s.x, s.wq, s.wk, None, s.gq, s.gk, EPS, s.rope, s.bufs[0], s.bufs[1], None, cd.SEND_MAJOR, None, None, None)
    # receiver: this rank's heads of every token
    for buf, hs in zip(s.received, s.hs):
        cd.a2a_unpack(s.mine, buf, hs, cd.RECV_MAJOR)
    cd.vmajor_select(s.Hp, s.N, s.d, TILE, s.own[2], s.v_prev, TAU, s.flags, s.idx, s.n_active, s.compact, s.cap, s.ws)
    return s.sent, s.own, s.flags, s.idx, s.n_active, s.compact


def _vmajor(s):
    H, N, d = s.H, s.N, s.d
    cd.vmajor_select(H, N, d, TILE, s.v, s.v_prev, TAU, s.flags, s.idx, s.n_active, s.compact, s.cap, s.ws)
    cd.vmajor_gather(H, N, d, TILE, s.q, s.idx, s.n_active, s.q_compact, s.cap)
    cd.vmajor_gather(H, N, d, TILE, s.k, s.idx, s.n_active, s.k_compact, s.cap)
    for compact, cache in zip((s.q_compact, s.k_compact, s.compact), s.caches):
        cd.vmajor_scatter(H, N, d, TILE, compact, s.idx, s.n_active, cache, s.cap)
    return s.flags, s.idx, s.n_active, s.compact, s.q_compact, s.k_compact, s.caches


def _tokens(s):
    cd.vmajor_token_metric(1, s.Ns, s.D, s.v, s.v_prev, s.metric)
    cd.vmajor_topk(1, s.Ns, s.metric, s.keep, s.idx, s.n_active)
    for t, compact, cache in zip((s.q, s.k, s.v), s.compact, s.caches):
        cd.vmajor_gather(1, s.Ns, s.D, 1, t, s.idx, s.n_active, compact, s.keep)
        cd.vmajor_scatter(1, s.Ns, s.D, 1, compact, s.idx, s.n_active, cache, s.keep)
    return s.metric, s.idx, s.n_active, s.compact, s.caches


def _back(s):
    cd.a2a_pack_hs(s.shape, s.y_hs, s.buf, cd.RECV_MAJOR)
    cd.a2a_unpack_seq(s.shape, s.buf, s.y_seq, cd.RECV_MAJOR)
    return s.buf, s.y_seq


_RUN = {"layer": _layer, "vfirst": _vfirst, "calls": _calls, "rank": _rank, "vmajor": _vmajor, "tokens": _tokens, "back": _back}


def run(state):
    return state.run(state)


def work(case):
    """Inputs read once, outputs written once (bf16: 2 bytes), 2 operations per multiply-add of the projections."""
    _, N, H, d, P = _sizes(case)
    D, kind = H * d, case["kind"]
    tensor, weights = N * D * 2, 3 * D * D * 2
    f = case.get("changed", 0.0)
    if kind == "back":
        return {"bytes": 3 * tensor, "flops": 0}                                   # y, buffer, y token-major
    if kind == "vmajor":
        return {"bytes": tensor * (2 + 2 * f + 6 * f), "flops": 0}                 # V twice, changed Q, K; compact x 3, caches x 3
    if kind == "tokens":
        kept = _kept_tokens(case) * D * 2
        return {"bytes": 2 * tensor / P + 2 * kept + 6 * kept, "flops": 3 * N // P * D}
    if kind == "rank":                                                             # x, sent x 3, received x 3, heads x 3, V before
        return {"bytes": tensor / P * (11 + f) + weights, "flops": 6 * N // P * D * D}
    outputs = 9 if kind == "calls" else 6                                          # token-major tensors too
    return {"bytes": tensor * (2 + outputs + f) + weights, "flops": 6 * N * D * D}


def tolerance(case):
    if case["kind"] in ("back", "vmajor"):
        return "exact"                              # copies, and a selection whose decisions are exact
    if case["kind"] == "tokens":
        return {"rel": 1e-5, "max": 1e-4}           # 32-bit sums; the kept tokens and what is copied are exact
    # one or two roundings to bf16 (2^-9 each, Q and K twice where the normalisation reads the rounded projection)
    return {"rel": 4e-3, "max": 2e-2}
