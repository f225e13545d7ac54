"""bench.py's argument checks that run before any GPU work."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args],
                          capture_output=True, text=True, timeout=120)


def test_more_than_one_gpu_is_refused_with_a_message():
    r = _run("--gpus", "2")
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def test_staleness_bound_is_refused_for_the_key_value_mix():
    r = _run("--config", "kv-uniform", "--staleness-bound", "0")
    assert r.returncode == 2
    assert "staleness-bound" in r.stderr


def test_unknown_dedup_mode_is_refused():
    r = _run("--dedup", "bucket")
    assert r.returncode == 2
    assert "--dedup" in r.stderr


def test_radix_dedup_moves_the_reduce_bytes_to_its_reduce_kernel():
    sys.path.insert(0, ROOT)
    import bench
    for n, U, M, D in ((212_992, 60_864, 0, 64), (4096, 1700, 1700, 16)):
        h = bench.kernel_bytes(n, U, M, D)
        r = bench.kernel_bytes(n, U, M, D, "radix")
        assert sum(h.values()) == sum(r.values())
        assert r["rsort_reduce"] == h["put_reduce"] and r["put_reduce"] == 0
        assert r["rsort_count"] == r["rsort_scatter"] == 0
    kv_h = bench.kernel_bytes_kv(1 << 19, 400_000, 1 << 19, 400_000, 4)
    kv_r = bench.kernel_bytes_kv(1 << 19, 400_000, 1 << 19, 400_000, 4, "radix")
    assert sum(kv_h.values()) == sum(kv_r.values()) and kv_r["rsort_reduce"] == kv_h["put_reduce"]


def test_a_gets_bytes_are_credited_to_its_two_kernels_together():
    # which of them copies the rows depends on the width and the batch size;
    # neither may show a rate for bytes the other moved
    sys.path.insert(0, ROOT)
    import bench
    for n, U, M, D in ((1 << 19, 400_000, 0, 4), (212_992, 60_864, 0, 64), (4096, 1700, 1700, 400)):
        b = bench.kernel_bytes(n, U, M, D)
        assert b["get"] == 8 * n + 12 * U + 4 * D * (U - M + n) + (4 * D + 16) * M
        prof = {k: (0.0, 0) for k in bench.KERNELS}
        prof.update(get_probe_gather=(0.2, 10), assign_new=(0.3, 10), put_probe=(0.1, 10), put_reduce=(0.4, 10))
        info = bench.kernel_info(prof, {k: 10 * v for k, v in b.items()})
        assert "gbps" not in info["get_probe_gather"] and "gbps" not in info["assign_new"]
        assert info["get"]["avg_us"] == 50.0 and info["get"]["alg_bytes_per_launch"] == b["get"]
        assert info["get"]["gbps"] == round(b["get"] / 50e-6 / 1e9, 1)
    assert bench.kernel_bytes_kv(100, 90, 100, 80, 4)["get"] == 8 * 100 + 12 * 90 + 16 * 190


def test_pipelined_steps_are_refused_at_bound_zero_and_for_the_key_value_mix():
    for extra in (("--staleness-bound", "0"), ("--config", "kv-zipf")):
        r = _run("--pipelined", *extra)
        assert r.returncode == 2
        assert "--pipelined" in r.stderr
