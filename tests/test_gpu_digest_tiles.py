"""build_digests at the edges of the tiles a wave takes: every element type, head dim and block size, blocks that do not
fill a wave's or a workgroup's share, partly filled last blocks, sequences of no and of one token; zeros of either sign,
infinities and NaNs (of equal elements the first stays, a NaN only in a block's first token).  Bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd import workload as W
from tests.gpu_harness import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S", [16, 32, 64])
@pytest.mark.parametrize("kind", [0, 1])
def test_digest_tiles(dtype, d, S, kind):
    Hkv, mb = 2, 37
    ctx = [mb * S, 36 * S + 1, 5 * S - 1, 17 * S + S // 2 + 3, 1, 0, S]
    rng = np.random.default_rng(d + S + kind)
    x = rng.standard_normal((len(ctx), Hkv, mb, S, d)).astype(np.float32)
    if kind == 0:
        special = np.array([0.0, -0.0, np.inf, -np.inf, np.nan], np.float32)
        at = rng.random(x.shape) < 0.2
        x[at] = special[rng.integers(0, 5, at.sum())]
        x[:, :, 3] = special[rng.integers(0, 2, x[:, :, 3].shape)]  # a block of zeros: only the signs differ
    K = W.to_storage(x, dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = torch.from_numpy(K.view(np.int16) if dtype == "bf16" else K).cuda().view(dt)
    lens = torch.tensor(ctx, dtype=torch.int32, device="cuda")
    p = B.make_problem(len(ctx), Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, mb, 4, lens, digest_kind=kind)
    if kind == 0:
        dig = torch.full((len(ctx), Hkv, mb, 2, d), 7.0, dtype=dt, device="cuda")
    else:
        dig = torch.full((len(ctx), Hkv, mb, d), 7.0, dtype=torch.float32, device="cuda")
    B.build_digests(p, dev, dig)
    got = to_np(dig)
    assert np.isfinite(W.storage_to_f32(got)).any()
    for b, n in enumerate(ctx):
        nb = (n + S - 1) // S
        for g in range(Hkv):
            rows = K[b, g].reshape(mb * S, d)
            want = oracle.digest(rows, n, S) if kind == 0 else oracle.digest_sum(rows, n, S)
            assert got[b, g, :nb].tobytes() == want.tobytes(), (b, g)
            assert (W.storage_to_f32(got[b, g, nb:]) == 7.0).all()  # rows beyond the sequence untouched
