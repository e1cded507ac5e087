"""The step with the selection in the attention launch, against the same step by separate calls, for rows of every number of keys per
lane that it is compiled for (2, 3, 4, 6, 8, 12 and 16: rows up to 512 times that), on the limits and one block beyond, in each of
its forms: one workgroup per pair, splits folded in the launch with the units dealt in ranges and in stride, heads that select for
themselves on the grid that keeps them together.

Every digest is there twice and the budget is odd, so that blocks share the score at its edge and the lower index has to win; a
sequence of no blocks, one that ends inside the first wave's keys and a full one are in the batch.  Scores and lists are equal bit for
bit.  Outputs: see test_gpu_fold_splits.py; here up to 80 tokens per wave."""
import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu

ROWS = [1024, 1025, 1536, 1537, 2048, 2049, 3072, 3073, 4096, 4097, 6144, 6145, 8192]


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("mb", ROWS)
@pytest.mark.parametrize("nsplit,per_head", [(1, 0), (2, 0), (9, 0), (1, 1)])
def test_selection_in_the_launch(dtype, d, mb, nsplit, per_head):
    Bn, Hkv, G, S, k, slots = 4, 2, 3, 16, 41, 200
    bf16, tdt = dtype == "bf16", torch.bfloat16 if dtype == "bf16" else torch.float32
    rand = dict(device="cuda", generator=torch.Generator(device="cuda").manual_seed(mb + d))
    ctx = torch.tensor([mb * S, 0, 37 * S - 5, (mb - 1) * S + 1], dtype=torch.int32, device="cuda")
    p = B.make_problem(Bn, G * Hkv, Hkv, d, S, B.BF16 if bf16 else B.F32, mb, k, ctx, per_head=per_head)
    q = torch.randint(-2, 3, (Bn, G * Hkv, d), **rand).to(tdt) / 4
    digest = torch.randint(-1, 2, (Bn, Hkv, mb, 1, d), **rand).expand(-1, -1, -1, 2, -1).to(tdt).contiguous()
    digest[..., 1, :] += 1
    half = mb // 2
    digest[:, :, half:2 * half] = digest[:, :, :half]
    kp, vp = (torch.randn(slots, S, d, **rand).to(tdt) for _ in range(2))
    table = torch.randint(-80, slots, (Bn, Hkv, mb), dtype=torch.int32, **rand).clamp_(min=-1)
    ho, hm = torch.randn(Bn, G * Hkv, d, **rand), torch.randn(Bn, G * Hkv, **rand)
    hl = torch.rand(Bn, G * Hkv, **rand) + 0.5
    rows, ws = G * Hkv if per_head else Hkv, B.alloc_workspace(p)

    def outputs():
        i32 = lambda *s: torch.full(s, -7, dtype=torch.int32, device="cuda")
        lists = i32(Bn, rows, k), i32(Bn, rows, k), i32(Bn, rows, k), i32(Bn, rows), i32(Bn, rows, k), i32(Bn, rows)
        return (torch.full((Bn, rows, mb), 7.0, device="cuda"), lists, torch.full((Bn, G * Hkv, d), float("nan"), dtype=tdt, device="cuda"),
                torch.full((Bn, G * Hkv), float("nan"), device="cuda"))

    scores, lists, out, lse = outputs()
    # (bf16 with d = 128 and one workgroup per pair scores short rows in the same launch, unless told not to)
    B.set_attn_mode(4 if bf16 and d == 128 else 0, nsplit, 0)
    try:
        B.layer_step(p, q, digest, table, kp, vp, slots, ho, hm, hl, scores, *lists, out, lse, ws)
    finally:
        B.set_attn_mode(0, 0, 0)
    scores2, lists2, want, want_lse = outputs()
    o, m, l = torch.empty(Bn, G * Hkv, d, device="cuda"), torch.empty(Bn, G * Hkv, device="cuda"), torch.empty(Bn, G * Hkv, device="cuda")
    B.score_blocks(p, q, digest, scores2, ws)
    B.select_topk(p, scores2, table, *lists2, ws)
    B.sparse_decode_attn(p, q, kp, vp, slots, lists2[1], lists2[2], lists2[3], o, m, l, ws)
    B.merge_partials(p, o, m, l, ho, hm, hl, want, want_lse)
    torch.cuda.synchronize()
    assert torch.equal(scores, scores2)
    for a, b in zip(lists, lists2):
        assert torch.equal(a, b)
    full = lists[0][0].long()   # the first sequence: as many blocks as the row holds, and ties at the edge of the budget
    kept = scores[0].gather(-1, full)
    edge = kept.min(-1, keepdim=True).values
    assert ((scores[0] == edge).sum(-1) > (kept == edge).sum(-1)).any()
    top = max(1.0, want.float().abs().max().item())
    vmax = vp.float().abs().max().item()
    bound = 2.0 ** -8 * (vmax + top) if bf16 else 1.2e-5 * top
    assert (out.float() - want.float()).abs().max().item() <= bound
    top = max(1.0, want_lse.abs().max().item())
    assert (lse - want_lse).abs().max().item() <= (2.0 ** -8 if bf16 else 1.2e-5 * top)
