"""The extension module that marshals calls refuses what the ctypes marshalling refuses, with the same exceptions, and what torch
throws while a tensor is looked into becomes a Python exception.  The calls run in a process of their own: an exception that
crossed into the interpreter's C frames would end it."""
import ctypes
import inspect
import json
import os
import subprocess
import sys

import pytest
import torch

from paper_2603_27138_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = """
import json, sys, warnings
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2603_27138_amd import binding as B
warnings.simplefilter("ignore")
p = B.Problem(1, 1, 1, 64, 16, 0, 4, 2, 0.0, 0, 0, 0, 0, 0, 0, 0x1000)
x, none8 = torch.zeros(2, 3), [None] * 8

class Looks:
    is_cuda = True
    def is_contiguous(self): return True
    def data_ptr(self): return 4096
    def numel(self): return "not a number"

def fake():
    with FakeTensorMode():
        y = torch.empty(4, device="cuda")
        return B.build_digests(p, y, y)

calls = dict(
    no_device=lambda: B.build_digests(p, None, None),
    vmap=lambda: torch.vmap(lambda y: B.recall_fetch(p, y, y, None, None, None, None, None, 0))(x),
    vmap_device=lambda: torch.vmap(lambda y: B.build_digests(p, y, y))(x),
    fake=fake,
    meta=lambda: B.build_digests(p, x.to("meta"), None),
    sparse=lambda: B.build_digests(p, x.to_sparse(), None),
    strided=lambda: B.recall_fetch(p, x.T, x, None, None, None, None, None, 0),
    host_tensor=lambda: B.build_digests(p, x, None),
    pageable=lambda: B.recall_fetch(p, x, x, None, None, None, None, None, 0),
    source_none=lambda: B.recall_fetch(p, None, None, None, None, None, None, None, 0),
    workspace_none=lambda: B.score_blocks(p, None, None, None, None),
    workspace_odd=lambda: B.score_blocks(p, None, None, None, Looks()),
    no_tensor=lambda: B.build_digests(p, 1, None),
    problem_none=lambda: B.build_digests(None, None, None),
    problem_bytes=lambda: B.build_digests(bytes(p), None, None),
    count_text=lambda: B.append_token(p, *none8, "x"),
    count_none=lambda: B.append_token(p, *none8, None),
    looks_like_one=lambda: B.build_digests(p, Looks(), Looks()),
    parameter=lambda: B.build_digests(p, torch.nn.Parameter(x), None),
)
for name in sys.argv[1:] or calls:
    try:
        calls[name]()
        got = ["none", ""]
    except Exception as e:
        got = [type(e).__name__, str(e)[:60]]
    print(json.dumps([name, *got]), flush=True)
"""

EXPECTED = {
    "vmap": "RuntimeError", "meta": "AssertionError", "sparse": "AssertionError", "strided": "AssertionError",
    "vmap_device": "AssertionError", "host_tensor": "AssertionError", "pageable": "AssertionError", "source_none": "AttributeError",
    "workspace_none": "AttributeError", "no_tensor": "AttributeError", "problem_none": "TypeError",
    "problem_bytes": "TypeError", "count_text": "ValueError", "count_none": "TypeError", "parameter": "AssertionError",
}
WITHOUT_GPU = {"no_device": "RuntimeError", "fake": "RuntimeError", "workspace_odd": "TypeError", "looks_like_one": "RuntimeError"}


def _run(names):
    env = dict(os.environ, PYTHONPATH=ROOT)
    res = subprocess.run([sys.executable, "-c", SCRIPT, *names], capture_output=True, text=True, cwd=ROOT, env=env, timeout=300)
    got = {n: (kind, text) for n, kind, text in (json.loads(ln) for ln in res.stdout.splitlines() if ln.startswith("["))}
    assert res.returncode == 0, (res.returncode, sorted(set(names) - set(got)), res.stderr[-500:])
    return got


@pytest.mark.skipif(torch.cuda.is_available(), reason="addresses that are none: only where nothing can be launched")
def test_refusals_are_python_exceptions():
    expected = {**EXPECTED, **WITHOUT_GPU}
    got = _run(list(expected))
    assert {n: kind for n, (kind, _) in got.items()} == expected
    assert "No HIP GPUs" in got["no_device"][1]
    assert got["host_tensor"][1] == "device tensors must be contiguous CUDA tensors"
    assert got["pageable"][1] == "need a CUDA tensor or a pinned CPU tensor"


def _arguments(fn):
    """A value of its own for every argument of a function of the binding."""
    args = {}
    for i, name in enumerate(inspect.signature(fn).parameters):
        if name == "p":
            args[name] = B.Problem(1, 2, 1, 64, 16, B.F32, 4, 2, 0.0, 0, 0, 0, 0, 0, 0, 0x1000)
        elif name == "n_slots":
            args[name] = 1000 + i
        elif name in ("host_k", "host_v", "src_k", "src_v"):
            args[name] = torch.zeros(16 + i, pin_memory=True)
        else:  # (staged: a whole number of tiles)
            args[name] = torch.zeros(2 * 16 * 64 * (1 + i), dtype=torch.uint8, device="cuda")
    return args


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["build_digests", "append_token", "score_blocks", "select_topk", "sparse_decode_attn",
                                  "sparse_decode_attn_static", "attn_partials", "attn_finish", "merge_partials", "periodic_recall",
                                  "recall_fetch", "recall_scatter", "layer_step"])
@pytest.mark.parametrize("form", ["plain", "subclass", "none"])
def test_both_marshallers_pass_the_same(name, form):
    """A call that is recorded (ctypes) and a call that is made (the extension module) hand the library the same arguments.  The
    module is bound to a function that keeps what it gets: nothing is launched."""
    class Sub(torch.Tensor):
        pass
    fn = getattr(B, name)
    args = _arguments(fn)
    optional = {"host_k", "host_v", "host_o", "host_m", "host_l", "scores", "lse", "o_b", "m_b", "l_b"}
    for key, v in args.items():
        if form == "subclass" and torch.is_tensor(v):
            args[key] = v.as_subclass(Sub)
        if form == "none" and key in optional:
            args[key] = None
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        (entry, cfunc, cargs), = B.prepare(fn, **args).calls
        want = [ctypes.addressof(args["p"])] + [getattr(a, "value", a) for a in cargs[1:]]
        got = []

        def keep(problem, *rest):
            got.append([ctypes.addressof(problem.contents), *rest])
            return 0

        callback = ctypes.CFUNCTYPE(ctypes.c_int, *cfunc.argtypes)(keep)
        table = {n: ctypes.cast(getattr(B.lib(), n), ctypes.c_void_p).value for n in B.EXPORTS}
        calls = B._calls or B._load_calls()
        calls.bind({**table, entry: ctypes.cast(callback, ctypes.c_void_p).value}, B.Problem, B._ptr, B._ptr_addressable, B._stream)
        try:
            fn(**args)
        finally:
            calls.bind(table, B.Problem, B._ptr, B._ptr_addressable, B._stream)
    assert got == [want] and want[-1] == side.cuda_stream


@pytest.mark.gpu
def test_batched_device_tensors_are_refused():
    p = B.Problem(1, 1, 1, 64, 16, B.F32, 4, 2, 0.0, 0, 0, 0, 0, 0, 0, 0x1000)
    with pytest.raises(RuntimeError):
        torch.vmap(lambda y: B.build_digests(p, y, y))(torch.zeros(2, 64, device="cuda"))
