"""build_digests where the rows of the batch could hold more keys than the memory-side cache (256 MiB), for batches that do
and batches that do not, and for more sequences than the lengths are looked at of: bit for bit what launches of a few
sequences each give, which stay below that size."""
import pytest
import torch

from paper_2603_27138_amd import binding as B

pytestmark = pytest.mark.gpu
LINE = 256 << 20


@pytest.mark.parametrize("dtype,d,S,kind", [("bf16", 128, 32, 0), ("bf16", 128, 64, 1), ("bf16", 64, 16, 0), ("bf16", 64, 64, 0),
                                            ("bf16", 64, 16, 1), ("f32", 128, 16, 0), ("f32", 64, 32, 0), ("f32", 128, 32, 1)])
@pytest.mark.parametrize("Bn,share", [(5, 1.0), (9, 0.05), (70, 0.9)])
def test_rows_beyond_the_memory_side_cache(dtype, d, S, kind, Bn, share):
    Hkv, tdt = 8, torch.bfloat16 if dtype == "bf16" else torch.float32
    block = Hkv * S * d * (2 if dtype == "bf16" else 4)
    mb = int(1.5 * LINE / (Bn * block)) + 1
    gen = torch.Generator(device="cuda").manual_seed(Bn + S)
    keys = torch.randn(Bn, Hkv, mb, S, d, dtype=tdt, device="cuda", generator=gen)
    assert keys.nbytes > LINE and keys.nbytes / Bn < LINE / 2
    ctx = torch.randint(int(0.9 * share * mb * S), int(share * mb * S) + 1, (Bn,), generator=gen, device="cuda", dtype=torch.int32)
    ctx[1] = 0
    ctx[-1] = int(share * mb * S)
    assert (int(ctx.sum()) * Hkv * d * keys.element_size() > LINE) == (share > 0.5)
    shape = (Bn, Hkv, mb, d) if kind else (Bn, Hkv, mb, 2, d)
    out_t = torch.float32 if kind else tdt
    whole, parts = (torch.full(shape, 7.0, dtype=out_t, device="cuda") for _ in range(2))

    def build(a, b, into):
        p = B.make_problem(b - a, Hkv, Hkv, d, S, B.BF16 if dtype == "bf16" else B.F32, mb, 4, ctx[a:b].clone(), digest_kind=kind)
        B.build_digests(p, keys[a:b], into[a:b])
        torch.cuda.synchronize()

    build(0, Bn, whole)
    step = 1 if Bn < 70 else 10
    for a in range(0, Bn, step):
        build(a, min(a + step, Bn), parts)
    as_int = torch.int32 if out_t == torch.float32 else torch.int16
    assert torch.equal(whole.view(as_int), parts.view(as_int))
    assert (whole[1] == 7.0).all() and not (whole[0, :, 0] == 7.0).all()
