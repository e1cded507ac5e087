"""The host worker's loops are compiled for several instruction sets and the widest one that the processor has runs.  Here the
narrower copies run the worker's own tests, and shapes at the edges of their blocks (heads, channels, tokens) are compared
with the attention in binary64: the logits (32-bit products of up to 256 channels, standard deviation 1) are good to 2^-19, so are
the weights, and the outputs are averages of values of unit variance."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("isa", [0, 1])
def test_narrower_copies_pass_the_workers_tests(tmp_path, isa):
    lib = str(tmp_path / f"libscout_host_{isa}.so")
    subprocess.run(["g++", "-O3", "-std=c++17", "-fPIC", "-shared", "-pthread", "-Wno-psabi", f"-DSCOUT_HOST_MAX_ISA={isa}", "-I",
                    os.path.join(ROOT, "include"), "-o", lib, os.path.join(ROOT, "paper_2603_27138_amd", "csrc", "host_worker.cpp")],
                   check=True)
    env = dict(os.environ, SCOUT_HOST_LIB=lib)
    res = subprocess.run([sys.executable, "-m", "pytest", "-x", "-q", "-p", "no:cacheprovider", "tests/test_host_worker.py",
                          "tests/test_host_isa.py::test_edges_of_the_blocks"], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, (res.stdout + res.stderr)[-3000:]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("G", [1, 2, 3, 5, 8, 9, 13, 16])
@pytest.mark.parametrize("d,S,ctx", [(8, 16, 33), (40, 7, 30), (64, 16, 48), (128, 64, 65), (248, 5, 23), (256, 32, 63)])
def test_edges_of_the_blocks(dtype, G, d, S, ctx):
    from paper_2603_27138_amd import host as H
    from paper_2603_27138_amd import workload as W
    rng = np.random.default_rng(G * d + S)
    B, Hkv = 1, 2
    mb = -(-ctx // S)
    make = lambda *s: W.to_storage(rng.standard_normal(s).astype(np.float32), dtype)
    q, K, V = make(B, Hkv * G, d), make(B, Hkv, mb, S, d), make(B, Hkv, mb, S, d)
    sel = np.tile(np.arange(mb, dtype=np.int32), (B, Hkv, 1))
    n = np.array([[mb, 0]], np.int32)
    o, m, l = np.ones((B, Hkv * G, d), np.float32), np.ones((B, Hkv * G), np.float32), np.ones((B, Hkv * G), np.float32)
    w = H.HostWorker(2)
    w.submit(H.HostProblem(B, Hkv * G, Hkv, d, S, 0 if dtype == "f32" else 1, mb, mb, 0.0), q, K, V, sel, n,
             np.array([ctx], np.int32), o, m, l)
    w.wait()
    w.close()
    f64 = lambda a: W.storage_to_f32(a).astype(np.float64)
    x = f64(q)[0, :G] @ f64(K)[0, 0].reshape(-1, d)[:ctx].T / np.sqrt(d)
    e = np.exp(x - x.max(1, keepdims=True))
    want = e @ f64(V)[0, 0].reshape(-1, d)[:ctx] / e.sum(1, keepdims=True)
    assert np.abs(o[0, :G] - want).max() < 2.0 ** -17
    lse = x.max(1) + np.log(e.sum(1))
    assert np.abs(m[0, :G].astype(np.float64) + np.log(l[0, :G].astype(np.float64)) - lse).max() < 2.0 ** -18
    assert not o[0, G:].any() and np.isneginf(m[0, G:]).all() and not l[0, G:].any()   # an empty list
