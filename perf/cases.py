"""Performance cases: what a decode loop, a prefill and a recall ask of the library, through the
public entry points of ``paper_2603_27138_amd.binding`` and ``.pipeline``.

A case is a dict of plain values:

  kind        "step"      one decode step: scout_layer_step on every layer, with append_token in front
                          of it where ``append`` is set
              "calls"     the same step by separate calls (score_blocks, select_topk, sparse_decode_attn,
                          merge_partials), as a caller runs it that works on the lists in between
              "digest"    build_digests over a prefilled batch
              "recall"    periodic_recall and the transfer of its tiles from pinned host memory
              "pipeline"  LayerAheadPipeline.step: Algorithm 1 with the host worker
  B, Hq, Hkv, d, S, dtype, k, p_host     as in scout_problem; p_host is the share of blocks in host memory
  ctx_lo, ctx_hi   tokens per sequence, uniform in [ctx_lo, ctx_hi]; one sequence has ctx_hi
  layers      layers of the model that a pass goes through, each with a cache of its own
  append, group_max, per_head, digest_kind, n_sink, n_tail     options, 0 where absent

Inputs follow paper_2603_27138_amd/workload.py (normal keys and values, 5 % of the blocks with keys
shifted along the group's query, shuffled pool slots), drawn on the GPU.  A layer is visited with two
queries in turn (cosine 0.98), as adjacent decode steps would.
"""
import math

import torch

from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd.pipeline import Layer, LayerAheadPipeline

HOST_THREADS = 5   # of each pipeline; several are alive at a time here, and idle workers spin before they sleep
PLANTED = 0.05     # share of blocks whose keys point along the group's query
Q_COS = 0.98       # cosine between the queries of two decode steps
RECALL_COS = 0.90  # cosine of the queries of two recalls to their common direction


def listed():
    c8b = dict(Hq=32, Hkv=8, d=128, S=32, dtype="bf16", k=64, p_host=0.4)
    c32b = dict(Hq=64, Hkv=8, d=128, S=32, dtype="bf16", k=64, p_host=0.5)
    return [
        # the smallest configuration of the repository: one sequence, one KV head, fp32; launches and
        # host time are all there is
        dict(name="tiny_f32", kind="step", B=1, Hq=4, Hkv=1, d=64, S=16, dtype="f32", k=16, p_host=0.25,
             ctx_lo=2048, ctx_hi=2048, layers=1),
        # one user: a single growing sequence through a few layers
        dict(name="one_sequence", kind="step", B=1, ctx_lo=20011, ctx_hi=20011, layers=4, append=1, **c8b),
        # a small batch of unequal, growing sequences
        dict(name="batch_8", kind="step", B=8, ctx_lo=24000, ctx_hi=32768, layers=4, append=1, **c8b),
        # the headline configuration: 16 sequences of 32k tokens
        dict(name="batch_16", kind="step", B=16, ctx_lo=32768, ctx_hi=32768, layers=4, **c32b),
        # few very long sequences, most of the cache on the host
        dict(name="long_context", kind="step", B=4, Hq=64, Hkv=8, d=128, S=32, dtype="bf16", k=128, p_host=0.75,
             ctx_lo=131072, ctx_hi=131072, layers=4),
        # a serving batch: 32 ragged, growing sequences of 4k to 64k tokens
        dict(name="ragged_32", kind="step", B=32, ctx_lo=4096, ctx_hi=65536, layers=2, append=1, **c32b),
        # every query head selects for itself
        dict(name="per_head", kind="step", B=8, ctx_lo=30000, ctx_hi=32768, layers=2, per_head=1, **c32b),
        # separate calls, importance by the maximum over the group, first and last block always kept
        dict(name="group_max_calls", kind="calls", B=8, ctx_lo=30000, ctx_hi=32768, layers=2, group_max=1, n_sink=1,
             n_tail=2, **c32b),
        # 64-channel heads and blocks of 16 tokens
        dict(name="heads_of_64", kind="step", B=8, Hq=32, Hkv=8, d=64, S=16, dtype="bf16", k=128, p_host=0.4,
             ctx_lo=8000, ctx_hi=16384, layers=4, append=1),
        # the end of a prefill: the digests of every block of a batch
        dict(name="prefill_digests", kind="digest", B=8, ctx_lo=16384, ctx_hi=32768, layers=1, **c32b),
        # a recall with a cache that is a little larger than the budget
        dict(name="recall", kind="recall", B=4, Hq=64, Hkv=8, d=128, S=32, dtype="bf16", k=64, p_host=0.84,
             ctx_lo=15000, ctx_hi=16384, layers=2),
        # the layer-ahead pipeline with the host's workers
        dict(name="pipeline", kind="pipeline", B=4, Hq=64, Hkv=8, d=128, S=32, dtype="bf16", k=64, p_host=0.05,
             ctx_lo=6000, ctx_hi=8192, layers=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "calls", "digest", "recall", "pipeline"], [10, 3, 2, 1, 1])[0]
    Hkv = rng.choice([1, 2, 4, 8])
    G = rng.choice([1, 2, 4, 4, 5, 8, 8, 16])
    d = rng.choice([128, 128, 64])
    S = rng.choice([16, 32, 32, 64])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    c = dict(kind=kind, Hkv=Hkv, Hq=G * Hkv, d=d, S=S, dtype=dtype, p_host=rng.choice([0.0, 0.25, 0.5, 0.75]))
    hi = _log_int(rng, 1000, 131072)
    if kind in ("recall", "pipeline"):
        hi = min(hi, 16384)
    lo = hi if rng.random() < 0.4 else rng.randint(max(1, hi // 8), hi)
    nb = (hi + S - 1) // S
    c["k"] = min(_log_int(rng, 16, 192), max(1, nb // 2))
    # the digest rows and tiles of the batch: at most what the largest listed case holds, an eighth of it
    # for the kinds and types that take longer per byte
    variant = rng.random()
    per_head = kind in ("step", "calls") and variant < 0.08
    cap = 16 * 8 * 32768 * 128 * 2 // (1 if dtype == "bf16" and kind in ("step", "digest") and not per_head else 8)
    per_seq = Hkv * hi * d * (2 if dtype == "bf16" else 4)
    c["B"] = min(_log_int(rng, 1, 48), max(1, cap // per_seq))
    c["ctx_lo"], c["ctx_hi"] = lo, hi
    c["layers"] = 1 if kind == "digest" else rng.randint(1, 4)
    while c["layers"] > 1 and c["layers"] * c["B"] * per_seq > 2 * cap:
        c["layers"] -= 1
    if kind == "step":
        c["append"] = int(rng.random() < 0.5)
    if kind in ("step", "calls"):
        if per_head:
            c["per_head"] = 1
        elif variant < 0.20:
            c["group_max"] = 1
        if rng.random() < 0.2:
            c["n_sink"], c["n_tail"] = 1, rng.randint(1, 3)
    if kind in ("step", "calls", "digest") and not c.get("group_max") and rng.random() < 0.12:
        c["digest_kind"] = 1
    if kind == "recall":
        c["p_host"] = max(0.0, 1.0 - 1.25 * c["k"] / nb)
    if kind == "pipeline":
        c["p_host"] = rng.choice([0.02, 0.05, 0.1])
    return c


# ------------------------------------------------------------------------------------------- inputs


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _max_tokens(case):
    return case["ctx_hi"] + (case["S"] if case.get("append") else 0)


def _max_blocks(case):
    return (_max_tokens(case) + case["S"] - 1) // case["S"]


class _Cache:
    """One layer: queries, digests, block table, pools, lists and outputs."""


def _layer(case, gen, ctx, p, queries, q_cos, want_blocks=False):
    Bn, Hq, Hkv, d, S = case["B"], case["Hq"], case["Hkv"], case["d"], case["S"]
    mb, dt, dev = _max_blocks(case), _torch_dtype(case), "cuda"
    rand = dict(generator=gen, device=dev)
    L = _Cache()
    base = torch.randn(Bn, Hq, d, **rand)
    L.q = [base.to(dt)] + [(q_cos * base + math.sqrt(1 - q_cos * q_cos) * torch.randn(Bn, Hq, d, **rand)).to(dt)
                           for _ in range(queries - 1)]
    u = base.view(Bn, Hkv, Hq // Hkv, d).sum(2)
    u = 3.0 * u / u.norm(dim=-1, keepdim=True)
    kb = torch.randn(Bn, Hkv, mb, S, d, dtype=dt, **rand)
    heavy = (torch.rand(Bn, Hkv, mb, 1, **rand) < PLANTED) * u[:, :, None, :]
    kb += heavy[:, :, :, None, :].to(dt)
    rows = (Bn, Hkv, mb)
    if case.get("digest_kind"):
        L.digest = torch.zeros(*rows, d, dtype=torch.float32, device=dev)
    else:
        L.digest = torch.zeros(*rows, 2, d, dtype=dt, device=dev)
    B.build_digests(p, kb, L.digest)
    nb = (ctx + S - 1) // S
    # every pair keeps the same share of its blocks resident; the pool has room for a full row of every pair
    beyond = torch.arange(mb, device=dev) >= nb[:, None, None]
    rank = (torch.rand(*rows, **rand) + 2 * beyond).argsort(-1).argsort(-1)
    keep = rank < ((1 - case["p_host"]) * nb).round()[:, None, None]
    at = keep.view(-1).nonzero().view(-1)
    at = at[torch.randperm(at.numel(), **rand)]
    n = at.numel()
    L.block_table = torch.full(rows, -1, dtype=torch.int32, device=dev)
    L.block_table.view(-1)[at] = torch.arange(n, dtype=torch.int32, device=dev)
    room = Bn * Hkv * (int((1 - case["p_host"]) * mb) + 1)
    spare = Bn * Hkv if case.get("append") else 0  # the slots of the blocks that the appends open
    L.n_slots = room + spare
    L.k_pool = torch.randn(L.n_slots, S, d, dtype=dt, **rand)
    L.v_pool = torch.randn(L.n_slots, S, d, dtype=dt, **rand)
    for i in range(0, n, 8192):
        L.k_pool[i:i + 8192][:min(8192, n - i)] = kb.view(-1, S, d)[at[i:i + 8192]]
    if spare:
        L.new_slot = (room + torch.arange(spare, dtype=torch.int32, device=dev)).view(Bn, Hkv)
        L.k_new = torch.randn(Bn, Hkv, d, dtype=dt, **rand)
        L.v_new = torch.randn(Bn, Hkv, d, dtype=dt, **rand)
        L.ctx0, L.ctx = ctx, ctx.clone()
    L.ho = L.hm = L.hl = None
    if case["p_host"] > 0:
        L.ho = 0.1 * torch.randn(Bn, Hq, d, **rand)
        L.hm = 2.0 + 0.3 * torch.randn(Bn, Hq, **rand)
        L.hl = torch.empty(Bn, Hq, device=dev).uniform_(50.0, 500.0, generator=gen)
    i32 = dict(dtype=torch.int32, device=dev)
    sel_rows, k = (Bn, Hq if case.get("per_head") else Hkv), case["k"]
    L.scores = torch.empty(*sel_rows, mb, device=dev)
    # the lists start as "nothing selected": the state of a fresh decode loop
    L.sel_all, L.sel_gpu, L.slot_gpu, L.sel_host = (torch.full((*sel_rows, k), -1, **i32) for _ in range(4))
    L.n_gpu, L.n_host = torch.zeros(sel_rows, **i32), torch.zeros(sel_rows, **i32)
    L.o, L.m, L.l = torch.empty(Bn, Hq, d, device=dev), torch.empty(Bn, Hq, device=dev), torch.empty(Bn, Hq, device=dev)
    L.out, L.lse = torch.empty(Bn, Hq, d, dtype=dt, device=dev), torch.empty(Bn, Hq, device=dev)
    if want_blocks:
        L.k_blocks = kb
    return L


def _problem(case, ctx, max_blocks):
    return B.make_problem(case["B"], case["Hq"], case["Hkv"], case["d"], case["S"],
                          B.BF16 if case["dtype"] == "bf16" else B.F32, max_blocks, case["k"], ctx,
                          **{f: case.get(f, 0) for f in ("n_sink", "n_tail", "group_max", "per_head", "digest_kind")})


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    mb, kind = _max_blocks(case), case["kind"]
    ctx = torch.randint(case["ctx_lo"], case["ctx_hi"] + 1, (case["B"],), generator=gen, device="cuda", dtype=torch.int32)
    ctx[0] = case["ctx_hi"]
    s = _State()
    s.kind, s.turn, s.S = kind, 0, case["S"]
    s.p = _problem(case, ctx, mb)
    s.ctx = ctx
    s.append, s.mean = bool(case.get("append")), bool(case.get("digest_kind"))
    queries, cos = (4, RECALL_COS) if kind == "recall" else (2, Q_COS)
    s.layers = [_layer(case, gen, ctx, s.p, queries, cos, kind in ("digest", "recall", "pipeline"))
                for _ in range(case["layers"])]
    s.ws = B.alloc_workspace(s.p)
    for L in s.layers:
        L.p = _problem(case, L.ctx, mb) if s.append else s.p
    if kind in ("recall", "pipeline"):
        for L in s.layers:
            rows = tuple(L.k_blocks.shape)
            L.src_k = torch.empty(rows, dtype=L.k_blocks.dtype, pin_memory=True).copy_(L.k_blocks)
            L.src_v = torch.empty(rows, dtype=L.k_blocks.dtype, pin_memory=True)
            L.src_v.copy_(L.k_blocks.flip(2))  # any values do
            del L.k_blocks
    if kind == "recall":
        for L in s.layers:
            lists = (case["B"], case["Hkv"], case["k"])
            L.recall_blk, L.recall_slot, L.evict_blk = (torch.empty(lists, dtype=torch.int32, device="cuda") for _ in range(3))
            L.n_recall = torch.empty(lists[:2], dtype=torch.int32, device="cuda")
    if kind == "pipeline":
        s.pipe = LayerAheadPipeline(case["B"], case["Hq"], case["Hkv"], case["d"], case["S"],
                                    B.BF16 if case["dtype"] == "bf16" else B.F32, mb, case["k"], ctx,
                                    [Layer(L.digest, L.block_table, L.k_pool, L.v_pool, L.n_slots, L.src_k, L.src_v)
                                     for L in s.layers], HOST_THREADS)
        # per layer the real query and the one predicted a layer ahead, for two decode steps
        s.real = [[L.q[t] for L in s.layers] for t in (0, 1)]
        s.pred = [[L.q[1 - t] for L in s.layers] for t in (0, 1)]
    return s


# --------------------------------------------------------------------------------------------- pass


def _lists(L):
    return dict(sel_all=L.sel_all, sel_gpu=L.sel_gpu, slot_gpu=L.slot_gpu, n_gpu=L.n_gpu, sel_host=L.sel_host, n_host=L.n_host)


def _run_step(s):
    turn = s.turn
    s.turn += 1
    for L in s.layers:
        if s.append:
            if turn % s.S == 0 and turn:  # the sequences ended: others of the same lengths take their places
                L.ctx.copy_(L.ctx0)
            B.append_token(L.p, L.ctx, L.k_new, L.v_new, L.new_slot, L.digest, L.block_table, L.k_pool, L.v_pool, L.n_slots)
        B.layer_step(L.p, L.q[turn & 1], L.digest, L.block_table, L.k_pool, L.v_pool, L.n_slots, L.ho, L.hm, L.hl, L.scores,
                     L.sel_all, L.sel_gpu, L.slot_gpu, L.n_gpu, L.sel_host, L.n_host, L.out, L.lse, s.ws)


def _run_calls(s):
    turn = s.turn
    s.turn += 1
    for L in s.layers:
        q = L.q[turn & 1]
        B.score_blocks(L.p, q, L.digest, L.scores, s.ws)
        B.select_topk(L.p, L.scores, L.block_table, L.sel_all, L.sel_gpu, L.slot_gpu, L.n_gpu, L.sel_host, L.n_host, s.ws)
        B.sparse_decode_attn(L.p, q, L.k_pool, L.v_pool, L.n_slots, L.sel_gpu, L.slot_gpu, L.n_gpu, L.o, L.m, L.l, s.ws)
        B.merge_partials(L.p, L.o, L.m, L.l, L.ho, L.hm, L.hl, L.out, L.lse)


def _run_recall(s):
    turn = s.turn
    s.turn += 1
    for L in s.layers:
        B.periodic_recall(L.p, L.q[turn & 3], L.digest, L.block_table, L.recall_blk, L.recall_slot, L.evict_blk, L.n_recall, s.ws)
        B.recall_fetch(L.p, L.src_k, L.src_v, L.recall_blk, L.recall_slot, L.n_recall, L.k_pool, L.v_pool, L.n_slots)


def run(s):
    if s.kind == "step":
        _run_step(s)
        outs = [dict(out=L.out, lse=L.lse, scores=L.scores, **_lists(L)) for L in s.layers]
        if s.append:  # what the append changed
            for L, o in zip(s.layers, outs):
                o.update(ctx=L.ctx, digest=L.digest, table=L.block_table, k_pool=L.k_pool, v_pool=L.v_pool)
        return outs
    if s.kind == "calls":
        _run_calls(s)
        return [dict(out=L.out, lse=L.lse, o=L.o, m=L.m, l=L.l, scores=L.scores, **_lists(L)) for L in s.layers]
    if s.kind == "digest":
        for L in s.layers:
            B.build_digests(L.p, L.k_blocks, L.digest)
        return [L.digest for L in s.layers]
    if s.kind == "recall":
        _run_recall(s)
        return [dict(blk=L.recall_blk, slot=L.recall_slot, evict=L.evict_blk, n=L.n_recall, table=L.block_table,
                     k_pool=L.k_pool, v_pool=L.v_pool) for L in s.layers]
    turn = s.turn & 1
    s.turn += 1
    s.pipe.step(s.real[turn], s.pred[turn])
    return [dict(out=b.out, lse=b.lse, sel_all=b.sel_all, sel_gpu=b.sel_gpu, n_gpu=b.n_gpu, sel_host=b.sel_host) for b in s.pipe.buf]


# --------------------------------------------------------------------------------------------- work


def work(case):
    """Each digest row, listed tile, query and host partial read once, each output written once."""
    Bn, Hq, Hkv, d, S, k = (case[f] for f in ("B", "Hq", "Hkv", "d", "S", "k"))
    es = 2 if case["dtype"] == "bf16" else 4
    mean_ctx = (case["ctx_hi"] + (Bn - 1) * (case["ctx_lo"] + case["ctx_hi"]) / 2) / Bn
    nb = mean_ctx / S
    rows = Bn * Hkv
    entry = 4 * d if case.get("digest_kind") else 2 * d * es
    if case["kind"] == "digest":
        keys = rows * mean_ctx * d
        return {"bytes": case["layers"] * (keys * es + rows * nb * entry), "flops": case["layers"] * 2 * keys}
    sel_rows = Bn * Hq if case.get("per_head") else rows
    tile = 2 * S * d * es
    listed_tiles = sel_rows * min(k, nb) * (1 - case["p_host"])
    heads = Hq / Hkv
    score = rows * nb * entry + Bn * Hq * d * es
    score_flops = rows * nb * 4 * d * (heads if case.get("group_max") or case.get("per_head") else 1)
    select = sel_rows * (nb * 8 + 4 * k * 4 + 8)  # a score and a table entry per block; the lists
    if case["kind"] == "recall":
        # a thirtieth of the budget returns per recall: the tiles come over the host link and go into the pool
        moved = 2 * rows * k / 30 * tile
        return {"bytes": case["layers"] * (score + select + moved), "flops": case["layers"] * score_flops}
    tiles = listed_tiles
    if case.get("per_head"):  # heads of one KV head that choose the same block need it once
        tiles = min(listed_tiles, rows * nb * (1 - case["p_host"]))
    attend = tiles * tile + Bn * Hq * (d * es + 4)
    if case["kind"] in ("calls", "pipeline"):
        attend += Bn * Hq * (d + 2) * 8  # the partial (o, m, l) leaves one call and enters the next
    if case["p_host"] > 0:
        attend += Bn * Hq * (d + 2) * 4
    if case["kind"] == "pipeline":  # the host's tiles
        attend += rows * min(k, nb) * case["p_host"] * tile
    if case.get("append"):
        attend += rows * d * es * 8
    attend_flops = listed_tiles * (1 if case.get("per_head") else heads) * S * d * 4
    return {"bytes": case["layers"] * (score + select + attend), "flops": case["layers"] * (score_flops + attend_flops)}


def tolerance(case):
    """Lists, tables, digests and moved tiles are exact.  Outputs: sums of 32-bit products for fp32; for
    bf16 the rounding of the softmax weights and of the output (2^-9 relative each)."""
    if case["kind"] in ("digest", "recall"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 5e-6}
    return {"rel": 8e-3, "max": 0.025}
