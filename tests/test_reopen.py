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


def test_closed_tables_memory_is_kept_bounded_and_given_back():
    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    def life(rows):
        t = mlkv.Table(64, rows)
        t.reserve(1000)
        held = free()
        t.close()
        return held

    slack = 16 << 20  # the driver's granularity, and what other code of the process allocates meanwhile
    mlkv.mlkv_trim()
    assert mlkv.mlkv_trim() == 0
    base = free()
    held = life(200_000)  # 51 MB of rows, 8 of index, and the scratch
    kept = base - free()
    assert 0 < kept <= (256 << 20) + slack
    assert free() < base - (40 << 20), "the table's memory was not kept"
    assert abs(life(200_000) - held) <= slack, "an equal table did not take the kept memory"
    for rows in (300_000, 400_000, 500_000, 600_000, 700_000):
        life(rows)
        assert base - free() <= (256 << 20) + slack
    given = mlkv.mlkv_trim()
    assert 0 < given <= 256 << 20
    assert mlkv.mlkv_trim() == 0 and abs(base - free()) <= slack
    log(f"[reopen] kept {kept >> 20} MiB, given back {given >> 20} MiB")


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
