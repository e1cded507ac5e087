"""The selection that leaves the host's job in pinned memory against the separate calls, bit for bit: every instance of the
selection kernel, whole and short sequences, budgets below and above the number of blocks, up to the largest; and the fold that
reads the host's partials from pinned memory against the one that reads them from the device."""
import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu


def _empty(*shape, dtype=torch.int32):
    return torch.full(shape, 77, dtype=dtype, device="cuda")


def _pinned(*shape, dtype=torch.int32):
    t = torch.empty(*shape, dtype=dtype, pin_memory=True)
    return t.fill_(-9)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 2, 128), ("f32", 16, 1, 64), ("bf16", 3, 3, 64)])
@pytest.mark.parametrize("mb,k", [(19, 40), (256, 64), (700, 9), (3000, 100), (4097, 1024)])
@pytest.mark.parametrize("per_head", [0, 1])
def test_select_ahead_is_score_and_select(dtype, Hq, Hkv, d, mb, k, per_head):
    Bn, S, tdt = 2, 16, torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(mb + k)
    q = torch.randn(Bn, Hq, d, device="cuda", generator=gen).to(tdt)
    lo = torch.randn(Bn, Hkv, mb, d, device="cuda", generator=gen)
    digest = torch.stack([lo, lo + 1.0], 3).to(tdt).contiguous()
    table = torch.where(torch.rand(Bn, Hkv, mb, device="cuda", generator=gen) < 0.5, -1, 3).to(torch.int32)
    ctx = torch.tensor([mb * S, mb * S // 3 + 1], dtype=torch.int32, device="cuda")
    p = B.make_problem(Bn, Hq, Hkv, d, S, B.F32 if dtype == "f32" else B.BF16, mb, k, ctx, per_head=per_head)
    rows = Hq if per_head else Hkv
    lists = lambda: [_empty(Bn, rows, k), _empty(Bn, rows, k), _empty(Bn, rows, k), _empty(Bn, rows), _empty(Bn, rows, k),
                     _empty(Bn, rows)]
    want, got, ws = lists(), lists(), B.alloc_workspace(p)
    scores, scores2 = (torch.empty(Bn, rows, mb, device="cuda") for _ in range(2))
    B.score_blocks(p, q, digest, scores, ws)
    B.select_topk(p, scores, table, *want, ws)
    job = _pinned(Bn, rows, k), _pinned(Bn, rows), _pinned(Bn, Hq, d, dtype=tdt)
    B.select_ahead(p, q, digest, table, scores2, *got, *job)
    torch.cuda.synchronize()
    assert torch.equal(scores, scores2)
    for a, b in zip(want, got):
        assert torch.equal(a, b)
    assert torch.equal(job[0], want[4].cpu()) and torch.equal(job[1], want[5].cpu()) and torch.equal(job[2], q.cpu())


def test_select_ahead_takes_only_addressable_buffers():
    ctx = torch.tensor([16], dtype=torch.int32, device="cuda")
    p = B.make_problem(1, 1, 1, 64, 16, B.F32, 1, 1, ctx)
    q, digest, table = torch.randn(1, 1, 64, device="cuda"), torch.randn(1, 1, 1, 2, 64, device="cuda"), _empty(1, 1, 1)
    lists = [_empty(1, 1, 1), _empty(1, 1, 1), _empty(1, 1, 1), _empty(1, 1), _empty(1, 1, 1), _empty(1, 1)]
    job = [_pinned(1, 1, 1), _pinned(1, 1), _pinned(1, 1, 64, dtype=torch.float32)]
    for i in range(3):
        bad = list(job)
        bad[i] = torch.empty(job[i].shape, dtype=job[i].dtype)   # pageable
        with pytest.raises(AssertionError):
            B.select_ahead(p, q, digest, table, torch.empty(1, 1, 1, device="cuda"), *lists, *bad)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 1, 128), ("f32", 16, 1, 64)])
def test_finish_reads_the_host_partials_from_pinned_memory(dtype, Hq, Hkv, d):
    Bn, S, mb, k, tdt = 2, 16, 40, 12, torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = torch.full((Bn,), mb * S, dtype=torch.int32, device="cuda")
    p = B.make_problem(Bn, Hq, Hkv, d, S, B.F32 if dtype == "f32" else B.BF16, mb, k, ctx)
    ws, n_slots = B.alloc_workspace(p), k
    q = torch.randn(Bn, Hq, d, device="cuda").to(tdt)
    kp, vp = (torch.randn(n_slots, S, d, device="cuda").to(tdt) for _ in range(2))
    sel = torch.arange(k, dtype=torch.int32, device="cuda").expand(Bn, Hkv, k).contiguous()
    n = torch.full((Bn, Hkv), k, dtype=torch.int32, device="cuda")
    host = torch.randn(Bn, Hq, d), torch.randn(Bn, Hq), torch.rand(Bn, Hq) * 100
    outs = []
    for parts, finish in (([t.cuda() for t in host], B.attn_finish), ([t.pin_memory() for t in host], B.attn_finish_ahead)):
        out, lse = torch.empty(Bn, Hq, d, dtype=tdt, device="cuda"), torch.empty(Bn, Hq, device="cuda")
        B.attn_partials(p, q, kp, vp, n_slots, sel, sel, n, ws)
        finish(p, *parts, out, lse, ws)
        outs.append((out, lse))
    torch.cuda.synchronize()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
