"""A batch of no sequences is nothing to do, for every entry point: no launch, no error (and no GPU needed to say so)."""
import ctypes

import pytest

from paper_2603_27138_amd import binding as B

X = ctypes.c_void_p(0x10000)   # aligned, and never looked at


def _calls(p):
    L, P, big = B.lib(), ctypes.byref(p), 1 << 30
    lists = [X] * 6
    return {
        "build_digests": lambda: L.build_digests(P, X, X, None),
        "append_token": lambda: L.append_token(P, *[X] * 8, 4, X, X, None),
        "score_blocks": lambda: L.score_blocks(P, X, X, X, X, big, None),
        "select_topk": lambda: L.select_topk(P, X, X, *lists, X, big, None),
        "scout_select_ahead": lambda: L.scout_select_ahead(P, X, X, X, X, *lists, X, X, X, None),
        "sparse_decode_attn": lambda: L.sparse_decode_attn(P, X, X, X, 4, *[X] * 7, big, None),
        "scout_attn_partials": lambda: L.scout_attn_partials(P, X, X, X, 4, X, X, X, X, big, None),
        "scout_attn_finish": lambda: L.scout_attn_finish(P, X, X, X, X, X, X, big, None),
        "merge_partials": lambda: L.merge_partials(P, *[X] * 8, None),
        "periodic_recall": lambda: L.periodic_recall(P, *[X] * 8, big, None),
        "recall_fetch": lambda: L.recall_fetch(P, *[X] * 7, 4, None),
        "recall_scatter": lambda: L.recall_scatter(P, X, 4, *[X] * 6, 4, None),
        "scout_layer_step": lambda: L.scout_layer_step(P, *[X] * 5, 4, X, X, X, X, *lists, X, X, X, big, None),
    }


@pytest.mark.parametrize("per_head", [0, 1])
@pytest.mark.parametrize("group_max,mb", [(0, 100), (0, 3000), (1, 3000), (0, 16384)])
@pytest.mark.parametrize("dtype,d", [(B.BF16, 128), (B.F32, 64)])
def test_no_sequences(dtype, d, group_max, mb, per_head):
    p = B.Problem(0, 8, 2, d, 16, dtype, mb, 32, 0.0, 0, 0, group_max, per_head, 0, 0, 0x10000)
    refused = {"periodic_recall": -2} if per_head else {}   # SCOUT_EUNSUPPORTED, whatever the batch
    for name, call in _calls(p).items():
        assert call() == refused.get(name, 0), name


def test_no_sequences_with_the_selection_as_a_launch_of_its_own():
    p = B.Problem(0, 8, 2, 128, 16, B.BF16, 100, 32, 0.0, 0, 0, 0, 0, 0, 0, 0x10000)
    for family in (1, 3, 4):
        try:
            B.set_attn_mode(family, 0, 0)
            assert _calls(p)["scout_layer_step"]() == 0
        finally:
            B.set_attn_mode(0, 0, 0)
