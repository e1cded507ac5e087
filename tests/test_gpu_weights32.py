"""Softmax weights stay binary32 for fp32 and for bf16 with d = 64, through every launch shape of the attention: the
exported partials and the merged outputs against a binary64 reference from the same lists.

Bound: a logit is a sum of d products in binary32, so its absolute error is at most d * 2^-24 * scale * sum |q k|, and a
weight's relative error is that; |q k| sums to at most 0.9 d here, which with scale = d^-1/2 gives 3.9e-6 (d = 64) and 7.8e-6 * 1.5
(d = 128) in the worst case.  The value sums add at most 64 tokens per wave and 64 partials (200 roundings, 1.2e-5).  Together
below 3e-5 of the largest value on outputs and on the logarithm of the weight sum.  Weights of 8 bits (2^-8 relative
each) miss it: 16 tokens in the list move an output by 3e-4 of the largest value, hundreds of tokens by 5e-5 and the logarithm by as much."""
import math

import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu
BOUND = 3e-5


def _reference(q, k_pool, v_pool, sel, slot, n, ctx, S):
    """(o normalised, log of the sum of exponentials) in binary64, per sequence and head."""
    Bn, Hq, d = q.shape
    Hkv = sel.shape[1]
    G = Hq // Hkv
    o = torch.zeros(Bn, Hq, d, dtype=torch.float64)
    lse = torch.full((Bn, Hq), -math.inf, dtype=torch.float64)
    q, k_pool, v_pool = (t.double().cpu() for t in (q, k_pool, v_pool))
    sel, slot, n, ctx = (t.cpu() for t in (sel, slot, n, ctx))
    for b in range(Bn):
        for g in range(Hkv):
            m = int(n[b, g])
            if m == 0:
                continue
            K, V = (pool[slot[b, g, :m].long()].reshape(m * S, d) for pool in (k_pool, v_pool))
            tok = (sel[b, g, :m, None].long() * S + torch.arange(S)).reshape(-1)
            x = q[b, g * G:(g + 1) * G] @ K[tok < ctx[b]].T / math.sqrt(d)
            lse[b, g * G:(g + 1) * G] = x.logsumexp(-1)
            o[b, g * G:(g + 1) * G] = x.softmax(-1) @ V[tok < ctx[b]]
    return o, lse


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("G,S,k,ctx", [(1, 16, 1, (16 * 40 - 3, 33)), (5, 32, 24, (32 * 70, 1)), (16, 64, 40, (64 * 90 + 17,)),
                                       (4, 16, 128, (16 * 200 + 1, 16 * 130))])
def test_weights_are_binary32(dtype, d, G, S, k, ctx):
    Hkv, Bn = 2, len(ctx)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(G + S)
    rand = dict(device="cuda", generator=gen)
    lens = torch.tensor(ctx, dtype=torch.int32, device="cuda")
    mb = max((c + S - 1) // S for c in ctx)
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, mb, k, lens)
    q = torch.randn(Bn, G * Hkv, d, **rand).to(tdt)
    slots = Bn * Hkv * mb
    k_pool, v_pool = (torch.randn(slots, S, d, **rand).to(tdt) for _ in range(2))
    table = torch.randperm(slots, **rand).int().view(Bn, Hkv, mb)
    digest = torch.zeros(Bn, Hkv, mb, 2, d, dtype=tdt, device="cuda")
    B.build_digests(p, k_pool[table.view(-1).long()].view(Bn, Hkv, mb, S, d).contiguous(), digest)
    f32, i32 = dict(dtype=torch.float32, device="cuda"), dict(dtype=torch.int32, device="cuda")
    sel_all, sel_gpu, slot_gpu, sel_host = (torch.empty(Bn, Hkv, k, **i32) for _ in range(4))
    n_gpu, n_host = torch.zeros(Bn, Hkv, **i32), torch.zeros(Bn, Hkv, **i32)
    slot_gpu.fill_(-1)
    scores = torch.empty(Bn, Hkv, mb, **f32)
    o, m, l = torch.empty(Bn, G * Hkv, d, **f32), torch.empty(Bn, G * Hkv, **f32), torch.empty(Bn, G * Hkv, **f32)
    out, lse = torch.empty(Bn, G * Hkv, d, dtype=tdt, device="cuda"), torch.empty(Bn, G * Hkv, **f32)
    ws = B.alloc_workspace(p)
    top = v_pool.float().abs().max().item()
    for mode in [(0, 0, 0), (0, 1, 0), (0, 2, 4), (0, 1, 16), (0, 3, 0)]:
        B.set_attn_mode(*mode)
        try:
            B.layer_step(p, q, digest, table, k_pool, v_pool, slots, None, None, None, scores, sel_all, sel_gpu, slot_gpu, n_gpu,
                         sel_host, n_host, out, lse, ws)
            B.sparse_decode_attn(p, q, k_pool, v_pool, slots, sel_gpu, slot_gpu, n_gpu, o, m, l, ws)
        finally:
            B.set_attn_mode(0, 0, 0)
        torch.cuda.synchronize()
        want, want_lse = _reference(q, k_pool, v_pool, sel_gpu, slot_gpu, n_gpu, lens, S)
        got = o.double().cpu()
        assert (got - want).abs().max().item() <= BOUND * top, mode
        assert ((m.double() + l.double().log()).cpu() - want_lse).abs().max().item() <= BOUND, mode
        half = 2.0 ** -8 if dtype == "bf16" else 0.0  # the output's own rounding: half a step of 2^-7 of the power of two below
        assert ((out.double().cpu() - want).abs() - half * want.abs()).max().item() <= BOUND * top, mode
        assert (lse.double().cpu() - want_lse).abs().max().item() <= BOUND, mode


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("mode", [(0, 0, 0), (0, 1, 0), (0, 2, 4)])
def test_infinite_values(dtype, d, mode):
    """A value that is infinite or no number gives what a positive weight times it gives, in its own channel only."""
    Bn, Hkv, G, S, k = 2, 2, 3, 16, 20
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rand = dict(device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    lens = torch.full((Bn,), k * S, dtype=torch.int32, device="cuda")
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, k, k, lens)
    q = torch.randn(Bn, G * Hkv, d, **rand).to(tdt)
    k_pool, v_pool = (torch.randn(Bn * Hkv * k, S, d, **rand).to(tdt) for _ in range(2))
    slot = torch.arange(Bn * Hkv * k, dtype=torch.int32, device="cuda").view(Bn, Hkv, k)
    sel = torch.arange(k, dtype=torch.int32, device="cuda").expand(Bn, Hkv, k).contiguous()
    n = torch.full((Bn, Hkv), k, dtype=torch.int32, device="cuda")
    inf = math.inf
    for at, ch, v in [(0, 3, inf), (7, 5, -inf), (2, 7, inf), (2 + k // 2, 7, -inf), (k - 1, 9, math.nan)]:
        v_pool[slot[:, :, at].long(), 4, ch] = v
    f32 = dict(dtype=torch.float32, device="cuda")
    o, m, l = torch.empty(Bn, G * Hkv, d, **f32), torch.empty(Bn, G * Hkv, **f32), torch.empty(Bn, G * Hkv, **f32)
    B.set_attn_mode(*mode)
    try:
        B.sparse_decode_attn(p, q, k_pool, v_pool, slot.numel(), sel, slot, n, o, m, l, B.alloc_workspace(p))
    finally:
        B.set_attn_mode(0, 0, 0)
    torch.cuda.synchronize()
    want, want_lse = _reference(q, k_pool, v_pool, sel, slot, n, lens, S)
    odd = [3, 5, 7, 9]
    assert torch.isposinf(want[..., 3]).all() and torch.isneginf(want[..., 5]).all() and torch.isnan(want[..., [7, 9]]).all()
    assert torch.isposinf(o[..., 3]).all() and torch.isneginf(o[..., 5]).all() and torch.isnan(o[..., [7, 9]]).all()
    rest = [c for c in range(d) if c not in odd]
    top = v_pool[torch.isfinite(v_pool)].float().abs().max().item()
    assert (o[..., rest].double().cpu() - want[..., rest]).abs().max().item() <= BOUND * top
    assert ((m.double() + l.double().log()).cpu() - want_lse).abs().max().item() <= BOUND


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
def test_weights_below_the_normal_range(dtype, d):
    """Weights of e^-88.5 = 2^-127.7: binary32 holds them to 22 bits, and large values make them count.  The rescaling between
    waves and splits flushes such factors, so the list is one unit.  (bf16 terms end at 2^-133: 2^-6 of the weight.)"""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ctx = torch.full((1,), 16, dtype=torch.int32, device="cuda")
    p = B.make_problem(1, 1, 1, d, 16, B.BF16 if dtype == "bf16" else B.F32, 1, 1, ctx, 1.0)
    q, k, v = torch.zeros(1, 1, d, dtype=tdt), torch.zeros(1, 16, d, dtype=tdt), torch.zeros(1, 16, d, dtype=tdt)
    q[0, 0, 0], k[0, 1:, 0], v[0, 1:] = 1, -88.5, 2.0 ** 100
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    zero, one = torch.zeros(1, 1, 1, dtype=torch.int32, device="cuda"), torch.ones(1, 1, dtype=torch.int32, device="cuda")
    o, m, l = torch.zeros(1, 1, d, device="cuda"), torch.zeros(1, 1, device="cuda"), torch.zeros(1, 1, device="cuda")
    B.sparse_decode_attn(p, q, k, v, 1, zero, zero, one, o, m, l, B.alloc_workspace(p))
    torch.cuda.synchronize()
    want = 15 * math.exp(-88.5) * 2.0 ** 100
    assert ((o.double() - want).abs() <= want * (2.0 ** -6 if dtype == "bf16" else 1e-4)).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("spread", [0.3, 2.0])
def test_error_no_larger_than_the_vector_alus(dtype, d, spread):
    """2-norm of the outputs' error against binary64, summed over lists of 64 to 1024 tokens with logits of the given standard
    deviation, of the matrix-core kernel and of the vector-ALU kernel on the same lists.  Both are sums of some 4000 rounding errors
    per case that differ in their order, so the two norms scatter by a few per cent of each other; a logit summed in one
    chain over 64 or 128 channels, or a rounded weight, shows as 2.2 to thousands of times the vector ALU's."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    square = {1: 0.0, 0: 0.0}
    for seed, (G, S, k) in enumerate([(4, 16, 4), (8, 32, 16), (16, 16, 64), (4, 32, 32), (8, 16, 16), (16, 32, 4)]):
        Bn, Hkv = 2, 8
        rand = dict(device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))
        lens = torch.full((Bn,), k * S, dtype=torch.int32, device="cuda")
        p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, k, k, lens)
        q = (spread * torch.randn(Bn, G * Hkv, d, **rand)).to(tdt)
        k_pool, v_pool = (torch.randn(Bn * Hkv * k, S, d, **rand).to(tdt) for _ in range(2))
        slot = torch.arange(Bn * Hkv * k, dtype=torch.int32, device="cuda").view(Bn, Hkv, k)
        sel = torch.arange(k, dtype=torch.int32, device="cuda").expand(Bn, Hkv, k).contiguous()
        n = torch.full((Bn, Hkv), k, dtype=torch.int32, device="cuda")
        want, _ = _reference(q, k_pool, v_pool, sel, slot, n, lens, S)
        f32 = dict(dtype=torch.float32, device="cuda")
        o, m, l = torch.empty(Bn, G * Hkv, d, **f32), torch.empty(Bn, G * Hkv, **f32), torch.empty(Bn, G * Hkv, **f32)
        for family in square:
            B.set_attn_mode(family, 0, 0)
            try:
                B.sparse_decode_attn(p, q, k_pool, v_pool, slot.numel(), sel, slot, n, o, m, l, B.alloc_workspace(p))
            finally:
                B.set_attn_mode(0, 0, 0)
            torch.cuda.synchronize()
            square[family] += ((o.double().cpu() - want).norm() / want.norm()).item() ** 2
    assert square[0] ** 0.5 <= 1.1 * square[1] ** 0.5, square
