"""Row assignment of few new keys (each block ranks its tiles' keys against
all new keys of the call), against the CPU oracle: at the limit where key
ranges take over, with more keys in one block than it ranks at a time (2048),
with more tiles to a block than it has threads. Bar: key -> row and rows
bit-exact. And the time of a put that inserts a few keys beside one that
inserts none."""
import numpy as np
import pytest
import torch

from paper_2504_01506_amd import mlkv
from _harness import Pair, dev_keys, log

pytestmark = pytest.mark.gpu

MULT = np.uint64(0x9E3779B97F4A7C15)


def _spread(ids):
    return np.asarray(ids, dtype=np.uint64) * MULT + np.uint64(5)


def _insert(pr, how, keys, rng, dim):
    rows = rng.normal(0, 0.01, size=(keys.size, dim)).astype(np.float32)
    if how == "get":
        pr.get(keys)
    elif how == "put":
        pr.put(keys, rows, 0.01, 1e-8)
    else:
        pr.upsert(keys, rows)
    assert pr.gpu.size == pr.ora.size
    assert np.array_equal(pr.gpu.lookup_rows(dev_keys(keys)).cpu().numpy(), pr.ora.lookup_rows(keys))


@pytest.mark.parametrize("how,n,new", [
    *((h, 4096, m) for h in ("put", "upsert") for m in (1, 614, 2048, 4096)),  # 64 tiles, 32 blocks
    *(("upsert", 30_000, m) for m in (16_384, 16_385)),  # the last direct put, the first by range
    *(("get", 8_192, m) for m in (1, 768, 769)),         # 128 tiles
    *(("get", 140_000, m) for m in (384, 385)),          # 547 tiles: two rounds of 512
])
@pytest.mark.parametrize("dim", [3, 36])
def test_few_new_keys(how, n, new, dim):
    rng = np.random.default_rng(n + new)
    old = 40_000
    pr = Pair(dim, old + new + 2)
    pr.get(_spread(np.arange(old)))
    ids = rng.integers(0, old, size=n)
    at = rng.permutation(n)
    ids[at[:new]] = old + rng.permutation(new)
    if new < n // 4:
        ids[at[new:2 * new]] = old + rng.integers(0, new, size=new)  # some of them again
    _insert(pr, how, _spread(ids), rng, dim)
    pr.compare_rows()
    pr.check_index()
    pr.close()


@pytest.mark.parametrize("how", ["put", "upsert"])
def test_more_new_keys_in_a_block_than_it_ranks_at_a_time(how):
    # 4096 put tiles of 1024, 512 assigning blocks: the new keys fill four
    # tiles of one block
    rng = np.random.default_rng(3)
    dim, n, old = 2, 4096 * 1024, 5_000
    pr = Pair(dim, old + 5000)
    pr.get(_spread(np.arange(old)))
    ids = rng.integers(0, old, size=(4096, 1024))
    ids[[5, 517, 1029, 4101 - 512]] = old + rng.permutation(4096).reshape(4, 1024)
    _insert(pr, how, _spread(ids.reshape(-1)), rng, dim)
    assert pr.gpu.size == old + 4096
    pr.compare_rows()
    pr.close()


def test_more_tiles_to_a_block_than_it_has_threads():
    # 262,656 get tiles of 256 positions, 512 assigning blocks of 512 threads
    n = 262_656 * 256
    t = mlkv.Table(1, 2000)
    t.get(torch.arange(1, 1001, device="cuda"), None)
    keys = torch.randint(1, 1001, (n,), device="cuda")
    keys[[300, n - 1]] = 5000
    t.get(keys, None)
    assert t.sync() == mlkv.MLKV_OK and t.size == 1001
    rows = t.lookup_rows(torch.tensor([1, 1000, 5000], device="cuda"))
    assert rows.tolist() == [0, 999, 1000]
    t.close()


def test_a_put_that_inserts_a_few_keys_takes_little_longer():
    n, old, times = 4096, 100_000, {}
    for new in (0, 600):
        t = mlkv.Table(4, old + 20 * 600)
        t.reserve(65_536)
        for s in range(0, old, 50_000):
            t.get(torch.arange(s, s + 50_000, device="cuda"), None)
        vals, us = torch.ones((n, 4), device="cuda"), []
        for step in range(12):
            keys = torch.randint(0, old, (n,), device="cuda")
            if new:
                keys[torch.randperm(n, device="cuda")[:new]] = torch.arange(old + step * new, old + (step + 1) * new,
                                                                            device="cuda")
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            t.put(keys, vals)
            b.record()
            torch.cuda.synchronize()
            us.append(a.elapsed_time(b) * 1e3)
        assert t.sync() == mlkv.MLKV_OK and t.size == old + 12 * new
        times[new] = float(np.median(us))
        t.close()
    log(f"[direct] put of {n} keys, us by new keys: {times}")
    # 45 us beside 24; 490 when blocks compared each tile's keys with all others
    assert times[600] < 8 * times[0]
