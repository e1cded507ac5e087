"""The one-launch step of pairs with little to read, against the same step by separate launches: every element type and
head dim, groups of 1, 5 and 16 heads, rows of one block, rows that end inside and at the end of a batch of the scoring
stream, empty sequences, budgets above the block count, and the largest budget and row that take the route.

Scores and lists are equal bit for bit.  Outputs: both add the same values in binary32 in another order, at most 64 tokens
per wave and 8 partials: 200 * 2^-24 = 1.2e-5 of the largest value; for bf16 the weights are rounded to bf16 against the
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
