"""The predicted query reaches the selection in the problem's own form: the selection and the host's worker see the same
values, and no kernel reads a tensor of another type or size as if it were the problem's."""
import types

import pytest
import torch

from paper_2603_27138_amd import pipeline as P


def _trigger(monkeypatch, q_pred, Bn=2, Hq=4, d=64, dtype=torch.bfloat16):
    """What _trigger hands to the selection."""
    seen = []
    monkeypatch.setattr(P.B, "select_ahead", lambda p, q, *rest: seen.append(q))
    names = "scores sel_all sel_gpu slot_gpu n_gpu sel_host n_host sel_host_h n_host_h".split()
    buf = types.SimpleNamespace(q_pred_h=torch.zeros(Bn, Hq, d, dtype=dtype), selected=types.SimpleNamespace(record=lambda: None),
                                **dict.fromkeys(names))
    layer = types.SimpleNamespace(digest=None, block_table=None)
    P.LayerAheadPipeline._trigger(types.SimpleNamespace(layers=[layer], buf=[buf], p=None), 0, q_pred)
    assert torch.equal(buf.q_pred_h, torch.zeros_like(buf.q_pred_h))   # only the selection writes the host's query
    return seen[0]


def test_the_query_itself(monkeypatch):
    q = torch.randn(2, 4, 64).bfloat16()
    assert _trigger(monkeypatch, q) is q


@pytest.mark.parametrize("shape,dtype", [((2, 4, 64), torch.float32), ((2, 4, 64), torch.float16), ((1, 4, 64), torch.bfloat16),
                                         ((4, 64), torch.bfloat16), ((64,), torch.float32), ((2, 1, 64), torch.float64)])
def test_another_form_is_what_a_copy_makes_of_it(monkeypatch, shape, dtype):
    q = torch.randn(*shape).to(dtype)
    got = _trigger(monkeypatch, q)
    want = torch.empty(2, 4, 64, dtype=torch.bfloat16).copy_(q)
    assert got.dtype == want.dtype and got.is_contiguous() and torch.equal(got, want)


@pytest.mark.parametrize("shape", [(3, 4, 64), (2, 4, 32), (1, 2, 4, 64), (2, 64, 4), (512,)])
def test_what_a_copy_refuses_is_refused_before_the_selection(monkeypatch, shape):
    with pytest.raises(RuntimeError):
        torch.empty(2, 4, 64).copy_(torch.zeros(*shape))
    calls = []
    monkeypatch.setattr(P.B, "select_ahead", lambda *a: calls.append(a))
    buf = types.SimpleNamespace(q_pred_h=torch.zeros(2, 4, 64), selected=None)
    layer = types.SimpleNamespace(digest=None, block_table=None)
    with pytest.raises(RuntimeError):
        P.LayerAheadPipeline._trigger(types.SimpleNamespace(layers=[layer], buf=[buf], p=None), 0, torch.zeros(*shape))
    assert not calls


def test_strided_queries_stay_refused():
    with pytest.raises(AssertionError):
        P._in_form_of(torch.zeros(4, 2, 64).transpose(0, 1), torch.zeros(2, 4, 64, dtype=torch.bfloat16))
