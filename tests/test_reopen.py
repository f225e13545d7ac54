"""Tables opened on the memory of closed ones: they start empty, and calls on
them match the CPU oracle, from one thread and from several."""
import threading

import numpy as np
import pytest
import torch

from paper_2504_01506_amd import mlkv
from _harness import Pair, log

pytestmark = pytest.mark.gpu

MULT = np.uint64(0x9E3779B97F4A7C15)


def _life(seed, cap, dim, bound=None):
    rng = np.random.default_rng(seed)
    pr = Pair(dim, cap, staleness_bound=bound)
    assert pr.gpu.size == 0
    _, _, sk, _ = pr.gpu.export(0)
    assert bool((sk == -1).all()), "a reopened table's index is not empty"
    for n in (500, 3000):
        keys = rng.integers(1, cap - 100, size=n).astype(np.uint64) * MULT
        if bound is None:
            pr.get(keys)
        else:
            pr.get_bounded(keys)
        pr.upsert(keys[: n // 2], rng.normal(size=(n // 2, dim)).astype(np.float32))
        pr.put(keys, rng.normal(0, 0.01, size=(n, dim)).astype(np.float32), 0.01, 1e-8)
    pr.compare_rows()
    pr.check_index()
    pr.close()


@pytest.mark.parametrize("dim", [5, 64])
def test_tables_reopened_on_released_memory(dim):
    for k in range(4):
        _life(k, 5000, dim, bound=1 if k == 2 else None)


def test_tables_opened_and_closed_from_several_threads():
    errors = []

    def work(seed):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(3):
                    t = mlkv.Table(8, 4000 + 100 * seed)
                    keys = torch.arange(1, 2001, dtype=torch.int64, device="cuda") * 7 + seed
                    vals = torch.full((2000, 8), float(seed * 10 + k), device="cuda")
                    out = torch.empty((2000, 8), device="cuda")
                    t.put(keys, vals)
                    t.get(keys, out)
                    assert t.sync() == mlkv.MLKV_OK and t.size == 2000
                    assert torch.equal(out, vals)
                    t.close()
        except BaseException as e:  # noqa: BLE001 - reported below
            errors.append((seed, e))

    threads = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
    log("[reopen] threads done")
