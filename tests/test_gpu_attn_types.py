"""The matrix-core attention for every element type and head dim, at the edges of its work split: groups of 1, 5
and 16 heads, fewer units than waves, partly filled last blocks and empty sequences, more than 64 units per wave,
several workgroups per pair, four and sixteen waves per workgroup; and the fused step on the same shapes.

Tolerances are the parity tests': binary32 sums of binary32 products for fp32 (1e-5 absolute on outputs of order 1),
for bf16 2e-2 absolute, which leaves room for rounded softmax weights; with d = 64 these are binary32, and
test_gpu_weights32.py holds the outputs to that."""
import numpy as np
import pytest
import torch

from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd import workload as W
from tests import harness
from tests.gpu_harness import Dev, to_np

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-5, "bf16": 2e-2}
TYPES = [("bf16", 64), ("f32", 64), ("f32", 128)]


def _check_partials(dev, res, cfg, mode):
    o, m, l = (t.cpu().numpy() for t in (dev.o, dev.m, dev.l))
    for (b, g), op in res.items():
        for h in range(cfg.G):
            hq = g * cfg.G + h
            wo, wm, wl_ = op.gpu_part[h]
            if wl_ == 0:
                assert (o[b, hq] == 0).all() and l[b, hq] == 0 and np.isneginf(m[b, hq]), mode
                continue
            assert np.abs(o[b, hq] - wo).max() <= TOL[cfg.dtype], (b, g, h, mode)
            assert abs(m[b, hq] + np.log(l[b, hq]) - (wm + np.log(wl_))) <= (1e-5 if cfg.dtype == "f32" else 2e-3) * max(1.0, abs(wm))


@pytest.mark.parametrize("dtype,d", TYPES)
@pytest.mark.parametrize("G,S,k,ctx", [(1, 16, 3, (33, 700)), (5, 32, 24, (0, 1, 1999)), (16, 64, 9, (64 * 20 + 17,)),
                                       (2, 64, 300, (64 * 330 + 5,))])
def test_attention_and_step(dtype, d, G, S, k, ctx):
    Hkv = 2
    cfg = W.shrink(W.tiny(), name=f"types-{dtype}-{d}-{G}-{S}", B=len(ctx), Hq=G * Hkv, Hkv=Hkv, d=d, S=S, dtype=dtype, ctx=ctx,
                   k=k, p_host=0.3)
    wl = W.generate(cfg)
    res = harness.run_all(wl)
    dev = Dev(wl)
    dev.set_digest_from_oracle(res)
    dev.set_host_partials_from_oracle(res)
    for mode in [(0, 0, 0), (0, 1, 0), (0, 3, 0), (0, 2, 4), (0, 1, 16)]:
        B.set_attn_mode(*mode)
        try:
            dev.set_selection_from_oracle(res)
            for t in (dev.o, dev.m, dev.l):
                t.fill_(float("nan"))
            dev.attn()
            _check_partials(dev, res, cfg, mode)
            dev.out.zero_()
            dev.layer_step()
        finally:
            B.set_attn_mode(0, 0, 0)
        sel, out = dev.sel_all.cpu().numpy(), W.storage_to_f32(to_np(dev.out)).astype(np.float64)
        excused = 0
        for (b, g), op in res.items():
            if not np.array_equal(sel[b, g], op.sel):
                assert harness.boundary_gap(op, cfg.k) < 1e-6
                excused += 1
                continue
            for h in range(G):
                assert np.abs(out[b, g * G + h] - op.out[h][0]).max() <= TOL[dtype], (b, g, h, mode)
        assert harness.few(excused, len(res))
