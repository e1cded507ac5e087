"""The fused step's own fold of a pair's splits against the fold by a launch of its own (the separate calls), from the
lists that the step wrote: split counts and groups on both sides of the line between the two, up to 63 splits folded
in the launch and 64 by the second launch, groups that divide the workgroup's threads and groups that do not, more splits
than one pass of the fold requests, shares that are empty.

The workspace starts as garbage, and the step is repeated on it: its counters must come from the step itself.

The separate attention deals the tokens to the waves in another order, so the partials differ as well as the order in
which they are added.  Binary32: at most 64 tokens per wave and 64 partials are added, each sum rounded once, and the
weights are rescaled a few times: 200 * 2^-24 = 1.2e-5 of the largest value.  bf16 (with d = 128; d = 64 keeps its weights
in binary32 and is held to the same bound): a weight is rounded to bf16 against the
maximum its wave knows, 2^-9 relative on either side, so 2^-8 on the weight sum (absolutely, on its logarithm) and 2^-8 of
the largest value vector element on the outputs, and one step of the output's type, 2^-8, more.
"""
import pytest
import torch

from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd import workload as W
from tests import harness
from tests.gpu_harness import Dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("G,k,nsplits", [(1, 8, (2, 3)), (3, 40, (2, 7, 33)), (4, 64, (16, 63, 64)), (8, 24, (2, 4, 9)),
                                         (16, 12, (2, 5, 64)), (16, 12, (3, 4, 7, 8, 33)), (8, 24, (3, 33))])
def test_fold_in_the_launch(dtype, d, G, k, nsplits):
    Hkv, S = 2, 16
    ctx = (S * 90 + 5, 0, 3, S * 41)
    cfg = W.shrink(W.tiny(), name=f"fold-{dtype}-{d}-{G}", B=len(ctx), Hq=G * Hkv, Hkv=Hkv, d=d, S=S, dtype=dtype, ctx=ctx, k=k,
                   p_host=0.3)
    wl = W.generate(cfg)
    dev = Dev(wl)
    dev.build_digests()
    dev.set_host_partials_from_oracle(harness.run_all(wl))
    bf16 = dtype == "bf16"
    vmax = max(abs(W.storage_to_f32(v)).max() for v in wl.V.values() if v.size)
    for nsplit in nsplits:
        B.set_attn_mode(0, nsplit, 0)
        try:
            dev.ws.fill_(0xFF)
            outs = []
            for _ in range(3):
                dev.out.fill_(float("nan"))
                dev.lse.fill_(float("nan"))
                dev.layer_step()
                outs.append((dev.out.clone(), dev.lse.clone()))
            dev.attn()
            dev.merge()
        finally:
            B.set_attn_mode(0, 0, 0)
        torch.cuda.synchronize()
        for out, lse in outs:
            assert torch.equal(out, outs[0][0]) and torch.equal(lse, outs[0][1]), nsplit
        out, want = outs[0][0].float(), dev.out.float()
        top = max(1.0, want.abs().max().item())
        assert (out - want).abs().max().item() <= (2.0 ** -8 * (vmax + top) if bf16 else 1.2e-5 * top), nsplit
        fin = torch.isfinite(dev.lse)
        assert torch.equal(torch.isfinite(outs[0][1]), fin)
        top = max(1.0, dev.lse[fin].abs().max().item())
        assert (outs[0][1] - dev.lse)[fin].abs().max().item() <= (2.0 ** -8 if bf16 else 1.2e-5 * top), nsplit


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("nsplit", [1, 3, 9])
def test_outputs_and_host_partials_may_start_at_any_element(dtype, d, nsplit):
    """The epilogues take channels two at a time: arrays that start one element behind an aligned address give the same bits."""
    cfg = W.shrink(W.tiny(), name=f"odd-{dtype}", B=2, Hq=8, Hkv=2, d=d, S=16, dtype=dtype, ctx=(16 * 90 + 5, 16 * 41), k=40, p_host=0.3)
    wl = W.generate(cfg)
    dev = Dev(wl)
    dev.build_digests()
    dev.set_host_partials_from_oracle(harness.run_all(wl))
    odd = lambda t: torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t)
    outs = []
    B.set_attn_mode(0, nsplit, 0)
    try:
        for shift in (lambda t: t.clone(), odd):
            ho, hm, hl, out, lse = (shift(t) for t in (dev.host_o, dev.host_m, dev.host_l, dev.out, dev.lse))
            B.layer_step(dev.p, dev.q, dev.digest, dev.block_table, dev.k_pool, dev.v_pool, dev.n_slots, ho, hm, hl, dev.scores, dev.sel_all,
                         dev.sel_gpu, dev.slot_gpu, dev.n_gpu, dev.sel_host, dev.n_host, out, lse, dev.ws)
            outs.append((out, lse))
    finally:
        B.set_attn_mode(0, 0, 0)
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
