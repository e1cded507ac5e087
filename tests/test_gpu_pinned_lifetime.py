"""Pinned host memory that kernels read or write belongs to them until they are done: a tensor that is dropped behind a call that
is still queued must not come back from the allocator of pinned memory for somebody else before that call has run.  The same holds for
device memory that a recall uses on the pipeline's copy stream."""
import gc

import pytest
import torch

from paper_2603_27138_amd import binding as B
from paper_2603_27138_amd import pipeline as P

pytestmark = pytest.mark.gpu

Bn, Hq, Hkv, d, S, mb, k = 1, 4, 1, 64, 16, 12, 4
BUSY = 400_000_000   # cycles that the stream is kept from starting the calls


def _i32(*s, **kw):
    return torch.zeros(s, dtype=torch.int32, **({"device": "cuda"} | kw))


def _problem():
    ctx = torch.full((Bn,), mb * S, dtype=torch.int32, device="cuda")
    return B.make_problem(Bn, Hq, Hkv, d, S, B.F32, mb, k, ctx), ctx


def _device_state():
    q, digest = torch.randn(Bn, Hq, d, device="cuda"), torch.randn(Bn, Hkv, mb, 2, d, device="cuda")
    kp, vp = torch.randn(mb, S, d, device="cuda"), torch.randn(mb, S, d, device="cuda")
    return q, digest, torch.arange(mb, dtype=torch.int32, device="cuda").view(Bn, Hkv, mb), kp, vp


def _pinned_again(sizes):
    """Addresses of fresh pinned tensors of these sizes, and enough of them to use up whatever lies on the free lists."""
    fresh = [torch.empty(n, dtype=torch.uint8, pin_memory=True) for n in sizes for _ in range(8)]
    return fresh, {t.data_ptr() for t in fresh}


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("call", ["select_ahead", "attn_finish_ahead", "append_token", "recall_fetch"])
def test_a_dropped_buffer_waits_for_the_stream(call, prepared):
    p, ctx = _problem()
    q, digest, table, kp, vp = _device_state()
    lists = [_i32(Bn, Hkv, k), _i32(Bn, Hkv, k), _i32(Bn, Hkv, k), _i32(Bn, Hkv), _i32(Bn, Hkv, k), _i32(Bn, Hkv)]
    ws, scores = B.alloc_workspace(p), torch.empty(Bn, Hkv, mb, device="cuda")
    out, lse = torch.empty(Bn, Hq, d, device="cuda"), torch.empty(Bn, Hq, device="cuda")
    pin = dict(pin_memory=True)
    blocks = (Bn, Hkv, mb, S, d)
    if call == "select_ahead":
        host = [_i32(Bn, Hkv, k, device="cpu", **pin), _i32(Bn, Hkv, device="cpu", **pin), torch.empty(Bn, Hq, d, **pin)]
        args = (p, q, digest, table, scores, *lists, *host)
    elif call == "attn_finish_ahead":
        host = [torch.zeros(Bn, Hq, d, **pin), torch.zeros(Bn, Hq, **pin), torch.zeros(Bn, Hq, **pin)]
        args = (p, *host, out, lse, ws)
    elif call == "append_token":   # of a full sequence: it is left as it is
        host = [torch.zeros(blocks, **pin), torch.zeros(blocks, **pin)]
        args = (p, ctx, q[:, :Hkv].contiguous(), q[:, :Hkv].contiguous(), _i32(Bn, Hkv), digest, table, kp, vp, mb, *host)
    else:                          # of nothing
        host = [torch.zeros(blocks, **pin), torch.zeros(blocks, **pin)]
        args = (p, *host, _i32(Bn, Hkv, k), _i32(Bn, Hkv, k), _i32(Bn, Hkv), kp, vp, mb)
    if call == "attn_finish_ahead":
        B.attn_partials(p, q, kp, vp, mb, *lists[1:4], ws)
    fn = getattr(B, call)
    replay = B.prepare(fn, *args) if prepared else None
    sizes, were = [t.numel() * t.element_size() for t in host], {t.data_ptr() for t in host}
    torch.cuda.synchronize()
    torch.cuda._sleep(BUSY)
    replay() if prepared else fn(*args)
    done = torch.cuda.Event()
    done.record()
    del host, args, replay
    fresh, now = _pinned_again(sizes)
    busy = not done.query()
    torch.cuda.synchronize()
    assert busy, "the stream was not kept busy for long enough"
    assert not were & now


def test_a_dropped_pipeline_waits_for_the_stream():
    _, ctx = _problem()
    q, digest, table, kp, vp = _device_state()
    table[0, 0, ::2] = -1
    kb, vb = (torch.randn(Bn, Hkv, mb, S, d).pin_memory() for _ in range(2))
    layer = P.Layer(digest, table, kp, vp, mb, kb, vb)
    pipe = P.LayerAheadPipeline(Bn, Hq, Hkv, d, S, B.F32, mb, k, ctx, [layer], n_threads=1,
                                filler=lambda i: torch.cuda._sleep(BUSY))
    want = [o.clone() for o in pipe.step([q], [q])]
    torch.cuda.synchronize()
    outs = pipe.step([q], [q])        # returns with the fold of the host's partials queued behind the filler
    done = torch.cuda.Event()
    done.record()
    b = pipe.buf[0]
    host = [b.sel_host_h, b.n_host_h, b.q_pred_h, b.ho_h, b.hm_h, b.hl_h]
    sizes, were = [t.numel() * t.element_size() for t in host], {t.data_ptr() for t in host}
    pipe.close()
    del pipe, b, host
    gc.collect()
    fresh, now = _pinned_again(sizes)
    for t in fresh:
        t.fill_(255)
    busy = not done.query()
    torch.cuda.synchronize()
    assert busy, "the stream was not kept busy for long enough"
    assert not were & now
    assert torch.equal(outs[0], want[0])


def test_a_dropped_pipeline_waits_for_its_copy_stream():
    _, ctx = _problem()
    q, digest, table, kp, vp = _device_state()
    table[0, 0, ::2] = -1
    kb, vb = (torch.randn(Bn, Hkv, mb, S, d).pin_memory() for _ in range(2))
    pipe = P.LayerAheadPipeline(Bn, Hq, Hkv, d, S, B.F32, mb, k, ctx, [P.Layer(digest, table, kp, vp, mb, kb, vb)], n_threads=1,
                                recall_every=1)
    digest[:, :, ::2] += 100.0        # the blocks in host memory are the important ones
    q.fill_(1.0)
    torch.cuda.synchronize()
    with torch.cuda.stream(pipe.copy_stream):
        torch.cuda._sleep(BUSY)
    pipe.step([q], [q])
    assert pipe.recalled_tiles > 0
    done, b = pipe.buf[0].arrived, pipe.buf[0]
    mine = [pipe.staged, pipe.tile_off, b.recall_blk, b.recall_slot, b.n_recall]
    sizes, were = [t.numel() * t.element_size() for t in mine], {t.data_ptr() for t in mine}
    pipe.close()
    del pipe, b, mine
    gc.collect()
    fresh = [torch.empty(n, dtype=torch.uint8, device="cuda") for n in sizes for _ in range(8)]
    busy = not done.query()
    torch.cuda.synchronize()
    assert busy, "the copy stream was not kept busy for long enough"
    assert not were & {t.data_ptr() for t in fresh}
