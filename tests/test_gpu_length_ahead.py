"""Digests that are requested before the sequence's length is known: whatever lies beyond the last block (here NaN patterns and
infinities) must leave no trace in scores, lists and outputs, for empty, short and full sequences, in every kernel that asks ahead
(scores of every kind, with as many heads as each of its instances takes: 4, 8, 16; the one-launch step of short rows) and on both
sides of the line in the number of pairs."""
import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("kind", ["sum", "mean", "max", "per_head"])
@pytest.mark.parametrize("Bn,Hkv,mb", [(3, 1, 200), (3, 43, 70), (3, 86, 70)])
@pytest.mark.parametrize("G", [4, 8, 11])
def test_scores_beyond_the_last_block(dtype, d, kind, Bn, Hkv, mb, G):
    S, tdt = 16, torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = torch.tensor([0, 5 * S + 3, mb * S], dtype=torch.int32, device="cuda")
    opts = dict(digest_kind=int(kind == "mean"), group_max=int(kind == "max"), per_head=int(kind == "per_head"))
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.F32 if dtype == "f32" else B.BF16, mb, 4, ctx, **opts)
    gen = torch.Generator(device="cuda").manual_seed(mb + d)
    q = torch.randn(Bn, G * Hkv, d, device="cuda", generator=gen).to(tdt)
    shape, t = ((Bn, Hkv, mb, d), torch.float32) if kind == "mean" else ((Bn, Hkv, mb, 2, d), tdt)
    clean = torch.rand(*shape, device="cuda", generator=gen).to(t)
    dirty = clean.clone()
    dirty[0], dirty[1, :, 6:] = float("nan"), float("inf")
    rows, ws = G * Hkv if kind == "per_head" else Hkv, B.alloc_workspace(p)
    got = []
    for dig in (clean, dirty):
        out = torch.full((Bn, rows, mb), 7.0, device="cuda")
        B.score_blocks(p, q, dig, out, ws)
        got.append(out)
    assert torch.equal(got[0], got[1])
    assert torch.isneginf(got[1][0]).all() and torch.isneginf(got[1][1, :, 6:]).all()
    assert torch.isfinite(got[1][1, :, :6]).all() and torch.isfinite(got[1][2]).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("Bn,Hkv", [(3, 1), (3, 100)])
def test_one_launch_step_beyond_the_last_block(dtype, d, Bn, Hkv):
    S, G, mb, k, tdt = 16, 4, 120, 8, torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = torch.tensor([0, 5 * S + 3, mb * S], dtype=torch.int32, device="cuda")
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.F32 if dtype == "f32" else B.BF16, mb, k, ctx)
    gen = torch.Generator(device="cuda").manual_seed(d)
    q = torch.randn(Bn, G * Hkv, d, device="cuda", generator=gen).to(tdt)
    clean = torch.rand(Bn, Hkv, mb, 2, d, device="cuda", generator=gen).to(tdt)
    dirty = clean.clone()
    dirty[0], dirty[1, :, 6:] = float("nan"), float("inf")
    kp, vp = (torch.randn(64, S, d, device="cuda", generator=gen).to(tdt) for _ in range(2))
    table = torch.randint(-1, 64, (Bn, Hkv, mb), device="cuda", generator=gen, dtype=torch.int32)
    got = []
    for dig in (clean, dirty):
        ws = torch.full((B.workspace_bytes(p),), 171, dtype=torch.uint8, device="cuda")
        i32 = lambda *s: torch.full(s, -7, dtype=torch.int32, device="cuda")
        lists = i32(Bn, Hkv, k), i32(Bn, Hkv, k), i32(Bn, Hkv, k), i32(Bn, Hkv), i32(Bn, Hkv, k), i32(Bn, Hkv)
        scores = torch.full((Bn, Hkv, mb), 7.0, device="cuda")
        out, lse = torch.zeros(Bn, G * Hkv, d, dtype=tdt, device="cuda"), torch.zeros(Bn, G * Hkv, device="cuda")
        B.layer_step(p, q, dig, table, kp, vp, 64, None, None, None, scores, *lists, out, lse, ws)
        assert bool((ws == 171).all())   # one launch: nothing went through the workspace
        got.append((scores, *lists, out, lse))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert torch.isneginf(got[0][0][0]).all() and (got[0][1][0] == -1).all()
