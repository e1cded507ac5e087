"""The one-launch step of pairs with little to read, against the same step by separate launches: every element type and
head dim, groups of 1, 5 and 16 heads, rows of one block, rows that end inside and at the end of a batch of the scoring
stream, empty sequences, budgets above the block count; then sizes on each limit of the route and one beyond it, where the
untouched workspace shows which route a call took (a launch of its own for the scores leaves them there).

Scores and lists are equal bit for bit.  Outputs: both add the same values in binary32 in another order, at most 64 tokens
per wave and 8 partials: 200 * 2^-24 = 1.2e-5 of the largest value; for bf16 with d = 128 the weights are rounded to bf16 against the
maximum a wave knows, 2^-9 relative on either side, and the output to bf16 (see test_gpu_fold_splits.py)."""
import pytest
import torch

from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd import workload as W
from tests import harness
from tests.gpu_harness import Dev

pytestmark = pytest.mark.gpu
NAMES = ("scores", "sel_all", "sel_gpu", "slot_gpu", "sel_host", "n_gpu", "n_host")


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("G,S,k,blocks", [(1, 16, 5, (1, 0, 3)), (5, 16, 16, (17, 16, 33, 8)), (16, 64, 2, (9, 31)),
                                          (4, 32, 8, (64, 63, 7)), (2, 16, 12, (100, 1))])
def test_one_launch_equals_separate_launches(dtype, d, G, S, k, blocks):
    Hkv = 2
    ctx = tuple(max(0, n * S - (i * 5 % S)) for i, n in enumerate(blocks))
    cfg = W.shrink(W.tiny(), name=f"small-{dtype}-{d}-{G}-{S}", B=len(ctx), Hq=G * Hkv, Hkv=Hkv, d=d, S=S, dtype=dtype, ctx=ctx,
                   k=k, p_host=0.3)
    wl = W.generate(cfg)
    dev = Dev(wl)
    dev.build_digests()
    dev.set_host_partials_from_oracle(harness.run_all(wl))
    got = {}
    for mode in [(0, 0, 0), (0, 2, 0)]:  # by the rule; two splits per pair, scored by a launch of their own
        B.set_attn_mode(*mode)
        try:
            for n in NAMES[:5]:
                getattr(dev, n).fill_(-7)
            dev.out.fill_(float("nan"))
            dev.layer_step()
        finally:
            B.set_attn_mode(0, 0, 0)
        got[mode] = {n: getattr(dev, n).clone() for n in NAMES + ("out", "lse")}
    a, b = got.values()
    for n in NAMES:
        assert torch.equal(a[n], b[n]), n
    vmax = max(abs(W.storage_to_f32(v)).max() for v in wl.V.values() if v.size)
    top = max(1.0, b["out"].float().abs().max().item())
    bound = 2.0 ** -8 * (vmax + top) if dtype == "bf16" else 1.2e-5 * top
    assert (a["out"].float() - b["out"].float()).abs().max().item() <= bound
    fin = torch.isfinite(b["lse"])
    assert torch.equal(torch.isfinite(a["lse"]), fin)
    top = max(1.0, b["lse"][fin].abs().max().item())
    assert (a["lse"] - b["lse"])[fin].abs().max().item() <= (2.0 ** -8 if dtype == "bf16" else 1.2e-5 * top)


def _one_launch(dtype, d, S, blocks, k, pairs):
    """Which calls take the one-launch route: little to read, or (bf16, d = 128) pairs that fill the chip."""
    row = 2 * d * (2 if dtype == "bf16" else 4)
    small = (blocks * row <= 128 << 10 and k * S <= 512 and (blocks + k * S) * row <= 288 << 10
             and (pairs <= 1024 or 2 * blocks >= k * S))
    fills = dtype == "bf16" and d == 128 and pairs >= 192 and blocks <= (2048 if pairs <= 256 else 1024)
    return small or fills


# blocks, S, k, sequences, one launch: on the limits (digests, listed tokens, both, pairs) and beyond
LIMITS = {
    ("bf16", 64): [(512, 16, 32, 2, 1), (513, 16, 32, 2, 0), (512, 16, 33, 2, 0), (40, 64, 8, 2, 1), (40, 64, 9, 2, 0),
                   (4, 16, 1, 512, 1), (4, 16, 1, 513, 0), (8, 16, 1, 513, 1)],
    ("bf16", 128): [(256, 16, 20, 2, 1), (257, 16, 19, 2, 0), (256, 16, 21, 2, 0), (64, 16, 32, 2, 1), (65, 16, 32, 2, 0),
                    (40, 16, 33, 2, 0), (257, 16, 33, 95, 0), (257, 16, 33, 96, 1), (4, 16, 1, 513, 1)],
    ("f32", 64): [(256, 16, 20, 2, 1), (257, 16, 19, 2, 0), (64, 16, 32, 2, 1), (65, 16, 32, 2, 0), (40, 32, 17, 2, 0),
                  (4, 16, 1, 512, 1), (4, 16, 1, 513, 0), (8, 16, 1, 513, 1)],
    ("f32", 128): [(128, 16, 10, 2, 1), (129, 16, 9, 2, 0), (128, 16, 11, 2, 0), (32, 16, 16, 2, 1), (33, 16, 16, 2, 0),
                   (4, 16, 1, 512, 1), (4, 16, 1, 513, 0), (8, 16, 1, 513, 1)],
}


@pytest.mark.parametrize("dtype,d,blocks,S,k,Bn,one", [(*t, *c) for t, cs in LIMITS.items() for c in cs])
def test_limits_of_the_route(dtype, d, blocks, S, k, Bn, one):
    Hkv, G, tdt = 2, 3, torch.bfloat16 if dtype == "bf16" else torch.float32
    assert _one_launch(dtype, d, S, blocks, k, Bn * Hkv) == bool(one)
    rand = dict(device="cuda", generator=torch.Generator(device="cuda").manual_seed(blocks + k))
    lens = torch.randint(0, blocks * S + 1, (Bn,), dtype=torch.int32, **rand)
    lens[0] = blocks * S
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, blocks, k, lens)
    slots = Bn * Hkv * blocks
    k_pool, v_pool = (torch.randn(slots, S, d, **rand).to(tdt) for _ in range(2))
    q = torch.randn(Bn, G * Hkv, d, **rand).to(tdt)
    place = torch.randperm(slots, **rand).int().view(Bn, Hkv, blocks)
    digest = torch.zeros(Bn, Hkv, blocks, 2, d, dtype=tdt, device="cuda")
    B.build_digests(p, k_pool[place.view(-1).long()].view(Bn, Hkv, blocks, S, d).contiguous(), digest)
    table = torch.where(torch.rand(Bn, Hkv, blocks, **rand) < 0.7, place, -1).int()
    ho, hm = torch.randn(Bn, G * Hkv, d, **rand), torch.randn(Bn, G * Hkv, **rand)
    hl = torch.rand(Bn, G * Hkv, **rand) + 0.5
    ws = B.alloc_workspace(p)
    got = []
    for mode in [(0, 0, 0), (0, 2, 0)]:  # by the rule; two splits per pair, scored by a launch of their own
        i32 = dict(dtype=torch.int32, device="cuda")
        lists = [torch.full((Bn, Hkv, k), -7, **i32) for _ in range(4)]
        n_gpu, n_host = torch.zeros(Bn, Hkv, **i32), torch.zeros(Bn, Hkv, **i32)
        out = torch.full((Bn, G * Hkv, d), float("nan"), dtype=tdt, device="cuda")
        lse = torch.full((Bn, G * Hkv), float("nan"), device="cuda")
        ws.fill_(0x5A)
        B.set_attn_mode(*mode)
        try:
            B.layer_step(p, q, digest, table, k_pool, v_pool, slots, ho, hm, hl, None, lists[0], lists[1], lists[2], n_gpu, lists[3],
                         n_host, out, lse, ws)
        finally:
            B.set_attn_mode(0, 0, 0)
        torch.cuda.synchronize()
        untouched = bool((ws == 0x5A).all())
        assert untouched == (bool(one) and mode[1] == 0), mode
        got.append((lists + [n_gpu, n_host], out.float(), lse))
    for a, b in zip(got[0][0], got[1][0]):
        assert torch.equal(a, b)
    (_, out, lse), (_, want, want_lse) = got
    top = max(1.0, want.abs().max().item())
    vmax = v_pool.float().abs().max().item()
    # (as above; bf16 with d = 64 keeps its weights in binary32, so that only the output's rounding is left: a step of 2^-7)
    bound = 2.0 ** -8 * (vmax + top) if (dtype, d) == ("bf16", 128) else (2.0 ** -7 if dtype == "bf16" else 0) * top + 1.2e-5 * top
    assert (out - want).abs().max().item() <= bound
    top = max(1.0, want_lse.abs().max().item())
    assert (lse - want_lse).abs().max().item() <= (2.0 ** -8 if (dtype, d) == ("bf16", 128) else 1.2e-5 * top)
