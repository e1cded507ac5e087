"""Head-wise scores in launches of few workgroups and of many: the same blocks give the same bits in a launch of a part of the batch
at a time and of the whole, where the first workgroups ask for their digests before they know the sequence's length in the one and
not in the other (up to 256 pairs, and beyond); and they are the binary64 scores rounded to binary32 (two summation orders in
binary64 differ by less than 2^-40 of the sum of magnitudes, so the rounded values by at most one step of 2^-23)."""
import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,line", [("bf16", 128, 256), ("bf16", 64, 256), ("f32", 64, 256), ("f32", 128, 256),
                                          ("bf16", 128, 1024), ("bf16", 64, 768), ("f32", 64, 1024), ("f32", 128, 1024),
                                          ("bf16", 64, 512), ("f32", 64, 512), ("f32", 128, 512)])
@pytest.mark.parametrize("G", [1, 3, 4, 5, 8, 9, 11, 16])   # up to 4, 8 and 16 heads run in instances of their own
@pytest.mark.parametrize("per_head", [0, 1])
def test_few_pairs_and_many(dtype, d, line, G, per_head):
    tdt, nb, S = (torch.bfloat16 if dtype == "bf16" else torch.float32), 19, 16   # one workgroup per pair
    Bn = line + 3
    gen = torch.Generator(device="cuda").manual_seed(7 + G)
    q = torch.randn(Bn, G, d, device="cuda", generator=gen).to(tdt)
    lo = torch.randn(Bn, 1, nb, d, device="cuda", generator=gen)
    digest = torch.stack([lo, lo + torch.rand(lo.shape, device="cuda", generator=gen)], 3).to(tdt).contiguous()
    ctx = torch.randint(0, nb * S + 1, (Bn,), device="cuda", generator=gen, dtype=torch.int32)

    def score(a, b):
        p = B.make_problem(b - a, G, 1, d, S, B.BF16 if dtype == "bf16" else B.F32, nb, 4, ctx[a:b], 0.0, group_max=1 - per_head,
                           per_head=per_head)
        out = torch.full((b - a, G if per_head else 1, nb), float("nan"), device="cuda")
        B.score_blocks(p, q[a:b], digest[a:b], out, B.alloc_workspace(p))
        return out

    many, few = score(0, Bn), torch.cat([score(0, line), score(line, Bn)])
    assert torch.equal(many, few)
    x = q.double()[:, :, None, :]
    each = torch.maximum(x * digest[:, :, :, 0].double(), x * digest[:, :, :, 1].double()).sum(-1)
    want = each if per_head else each.amax(1, keepdim=True)
    beyond = (torch.arange(nb, device="cuda")[None] >= (ctx[:, None] + S - 1) // S)[:, None].expand_as(many)
    assert torch.isneginf(many[beyond]).all()
    assert ((many.double() - want)[~beyond].abs() <= 2.0 ** -23 * want[~beyond].abs() + 1e-9).all()
