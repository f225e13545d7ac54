"""The first calls of a process: opening a table loads the device code its
calls run (a code object for each row map, one for tiered tables, one with
the array of the allocation-free get), so that a first put or lookahead, also
under stream capture, loads nothing. Each check runs in a process of its own,
where nothing is loaded yet."""
import os
import subprocess
import sys

import pytest

from _harness import log

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _child(body):
    head = "import time, numpy as np, torch\nfrom paper_2504_01506_amd import mlkv\ntorch.cuda.set_device(0)\n"
    r = subprocess.run([sys.executable, "-c", head + body], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


def test_first_put_of_each_row_map_loads_no_code():
    # a first put takes about 45 us, with its code object to load 450
    out = _child("""
k = torch.arange(1, 4097, device="cuda")
for dim in (3, 16, 32, 64, 128, 256, 512, 1024):
    t = mlkv.Table(dim, 8192)
    t.reserve(4096)
    o, g = torch.empty((4096, dim), device="cuda"), torch.ones((4096, dim), device="cuda")
    t.get(k, o)
    torch.cuda.synchronize()
    a = time.perf_counter()
    t.put_grad(k, g, 0.01, 1e-8)
    torch.cuda.synchronize()
    print((time.perf_counter() - a) * 1e6)
    assert t.sync() == mlkv.MLKV_OK and t.size == 4096
""")
    us = sorted(float(x) for x in out.split())
    log(f"[first] first puts, us: {us}")
    assert len(us) == 8 and us[3] < 200.0


def test_first_calls_under_stream_capture():
    # one replay each: a replayed call is the one call that was captured
    _child("""
dim, k = 100, torch.arange(1, 2001, device="cuda")
t = mlkv.Table(dim, 4096)
t.reserve(4096)
o, g = torch.empty((2000, dim), device="cuda"), torch.ones((2000, dim), device="cuda")
t.get(k, o)
want = o.clone()
assert t.sync() == mlkv.MLKV_OK
o.zero_()
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    assert mlkv.mlkv_get_noalloc(t.h, k, 2000, o) == mlkv.MLKV_OK
    t.put_grad_sgd(k, g, 0.5)
graph.replay()
torch.cuda.synchronize()
assert t.sync() == mlkv.MLKV_OK and torch.equal(o, want)
t.get(k, o)
assert t.sync() == mlkv.MLKV_OK and torch.equal(o, want - 0.5)
""")
