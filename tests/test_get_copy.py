"""Gets at the edges of the rule that says which kernel copies their rows
(with the probe, 4, 8 or 16 lanes a row, or apart), against the CPU oracle:
present and new keys, keys a lookahead recorded, blocked positions, outputs
off 16 bytes and outputs large enough to go around the caches. Bar: rows and
key -> row bit-exact, nothing written outside the buffer."""
import numpy as np
import pytest
import torch

from paper_2504_01506_amd import mlkv
from _harness import Pair, dev_keys

pytestmark = pytest.mark.gpu

MULT = np.uint64(0x9E3779B97F4A7C15)
TILES = 256 * torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 1 << 16
SIZES = {5: (63, 1000), 16: (64, 700, 530_000), 17: (TILES, TILES + 1), 32: (TILES, TILES + 1, 270_000),
         33: (TILES, TILES + 1), 64: (TILES + 1, 140_000, 6 * TILES, 6 * TILES + 1), 65: (TILES + 1,)}


@pytest.mark.parametrize("dim,n", [(d, n) for d, ns in SIZES.items() for n in ns])
def test_rows_are_copied_alike_on_every_route(dim, n):
    rng = np.random.default_rng(dim + n)
    pr = Pair(dim, 130_000)
    pr.prefill(np.sort(np.arange(1, 50_001).astype(np.uint64) * MULT))
    guard = np.float32(-7.25)
    buf = torch.full((n * dim + 8,), float(guard), device="cuda")
    for step, shift in enumerate((0, 1, 2)):
        ids = rng.integers(1, 50_001 + 20_000 * step, size=n)  # from the second on, some are new
        keys = ids.astype(np.uint64) * MULT
        if step == 2:
            pr.lookahead(keys[: n // 2 + 1])  # half of the positions skip the probe
        out = buf[shift:shift + n * dim].view(n, dim)
        pr.gpu.get(dev_keys(keys), out)
        rc, want = pr.ora.get(keys)
        assert rc == 0 and pr.gpu.sync() == mlkv.MLKV_OK and pr.gpu.size == pr.ora.size
        pr.compare_get(keys, out.cpu().numpy(), want)
        edge = torch.cat([buf[:shift], buf[shift + n * dim:]])
        assert bool((edge == float(guard)).all()), "written outside the buffer"
        buf.fill_(float(guard))
    pr.check_index()
    pr.close()


@pytest.mark.parametrize("dim,n", [(4, 500), (16, 500), (16, 530_000), (32, TILES + 1), (32, 270_000),
                                   (64, TILES + 1), (64, 140_000), (64, 6 * TILES + 1)])
def test_blocked_positions_on_every_route(dim, n):
    rng = np.random.default_rng(dim * 3 + n)
    pr = Pair(dim, 60_000, staleness_bound=0)
    pr.prefill(np.sort(np.arange(1, 40_001).astype(np.uint64) * MULT))
    for hi in (20_000, 59_000):  # the second get: keys of the first are blocked, others present or new
        bl = pr.get_bounded(rng.integers(1, hi, size=n).astype(np.uint64) * MULT)
    assert bl.any() and not bl.all()
    pr.compare_staleness()
    pr.close()
