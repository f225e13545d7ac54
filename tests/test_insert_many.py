"""Puts and gets that insert a million keys and more in one call, against the
CPU oracle: key ranges that hold more keys than a block ranks in LDS (3072; at
2^20 new keys some of a put's 512 ranges do, at 2^22 every one), a dense
cluster of keys among spread ones, keys repeated so that an upsert's last
position matters, and a call of that size that does not fit."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2504_01506_amd import mlkv
from _harness import Pair, dev, dev_keys

pytestmark = pytest.mark.gpu

MULT = np.uint64(0x9E3779B97F4A7C15)


def _keys(rng, new, cluster):
    keys = np.arange(1, new + 1).astype(np.uint64) * MULT
    if cluster:  # most of them within a narrow interval
        keys[new // 4:] = np.uint64(1 << 40) + np.arange(new - new // 4, dtype=np.uint64)
    keys = rng.permutation(keys)
    again = rng.choice(keys, size=new // 8)  # later positions of some, in other tiles
    return np.concatenate([keys, again])


@pytest.mark.parametrize("how", ["get", "put", "upsert"])
@pytest.mark.parametrize("new,cluster", [(1 << 20, False), (1 << 20, True), (1 << 22, False)])
def test_a_call_that_inserts_every_key(how, new, cluster):
    rng = np.random.default_rng(new + cluster)
    keys = _keys(rng, new, cluster)
    rows = rng.normal(0, 0.01, size=(keys.size, 2)).astype(np.float32)
    pr = Pair(2, new + 100)
    if how == "get":
        pr.get(keys)
    elif how == "put":
        pr.put(keys, rows, 0.01, 1e-8)
    else:
        pr.upsert(keys, rows)
    assert pr.gpu.size == pr.ora.size == new
    assert np.array_equal(pr.gpu.lookup_rows(dev_keys(keys)).cpu().numpy(), pr.ora.lookup_rows(keys))
    pr.compare_rows()
    pr.close()


@pytest.mark.parametrize("how", ["put", "upsert"])
def test_a_call_that_does_not_fit_leaves_the_table_as_it_was(how):
    rng = np.random.default_rng(4)
    new = 1 << 20
    keys = _keys(rng, new, False)
    rows = rng.normal(0, 0.01, size=(keys.size, 2)).astype(np.float32)
    pr = Pair(2, new - 1)
    pr.upsert(keys[:1000], rows[:1000])
    kd, rd = dev_keys(keys), dev(rows)
    if how == "put":
        pr.gpu.put_grad(kd, rd, 0.01, 1e-8)
        assert pr.ora.put_grad(keys, rows, 0.01, 1e-8) == O.EFULL
    else:
        pr.gpu.put(kd, rd)
        assert pr.ora.put(keys, rows) == O.EFULL
    assert pr.gpu.sync() == mlkv.MLKV_EFULL and pr.gpu.size == 1000
    pr.compare_rows()
    pr.check_index()
    fits = keys[: new // 2]
    pr.upsert(fits, rows[: fits.size])  # the failed call left no key and no position behind
    pr.compare_rows()
    pr.close()
