"""Host-side checks of bench.py: the one-GPU contract, the plan's byte
accounting against the paper's per-pass traffic, and the counter summaries it
reads its traffic figure from."""
import json
import os
import re
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def _summary(key):
    path = os.path.join(ROOT, "profiles", bench.COUNTERS_FILES[key])
    m = re.search(r"```json\s*(\{.*?\})\s*```", open(path).read(), flags=re.S)
    return json.loads(m.group(1))


@pytest.mark.parametrize("key", sorted(bench.COUNTERS_FILES), ids=lambda k: "-".join(k))
def test_counter_summaries_are_well_formed(key):
    """The committed summaries carry the FETCH_SIZE / WRITE_SIZE calibration
    and a traffic figure near the counted bytes (a state that stays in the caches
    moves less; rows of a run are also evicted and read again a little)."""
    kernel, workload, proxy = key
    d = _summary(key)
    assert (d["kernel"], d["workload"], d["proxy"]) == key
    assert d["fetch_scale"] == pytest.approx(2.0, rel=1e-3)
    assert d["write_scale"] == pytest.approx(1.0, rel=1e-3)
    ratio = d["bytes_per_launch"] / d["alg_bytes_per_launch"]
    assert (0.0 < ratio < 1.05) if workload == "small" else (0.9 <= ratio < 1.1)
    if kernel == "pass_kernel" and workload == "headline":
        # P'(16 + 16 D) bytes a pass, with the shared moment P'(24 + 8 D)
        base, row = (16, 16) if proxy == "local" else (24, 8)
        assert 20 < (d["alg_bytes_per_launch"] / 25_000_000 - base) / row <= 32
    if kernel == "seg_step_kernel":   # 32 bytes per element-commit with post-commit pulls
        assert d["alg_bytes_per_launch"] == pytest.approx(32 * 25_000_000, rel=1e-5)
    assert d["valu_instrs_per_launch"] > 0


def test_traffic_is_withheld_for_other_sources(monkeypatch):
    """The counter figures are only reported while the kernel sources hash to
    the value recorded with the counters."""
    monkeypatch.setattr(bench, "kernel_hash", lambda: "0" * 16)
    for key in bench.COUNTERS_FILES:
        assert bench.measured_counters(*key) is None
    assert bench.measured_counters("short_run_kernel", "tiny", "local") is None


def test_run_plan_counts_what_a_run_moves():
    """The byte count of a run's launches on a device of 256 compute units: a
    short vector moves each worker's rows once a launch; a longer one at most a
    row each way per commit, fewer than its passes, and with as many workers as
    slots only the first and last of each; the shared moment, half of each."""
    import oracle as O
    from paper_1805_08469_amd.workloads import WORKLOADS
    dev = dict(cus=256, lds=160 << 10)
    wl = WORKLOADS["tiny"]
    worker, _ = O.schedule(wl.n, wl.T, wl.law, wl.law_p0, wl.law_p1, seed=wl.seed)
    p = bench.run_plan(wl, worker, False, False, **dev)
    assert (p["launches"], p["short"]) == (-(-wl.T // 993), -(-wl.T // 993))
    assert p["bytes"] == wl.P * p["launches"] * (16 + 2 * 8 * wl.n)
    wl = WORKLOADS["headline"]
    worker, _ = O.schedule(wl.n, wl.T, wl.law, wl.law_p0, wl.law_p1, seed=wl.seed)
    p, q = (bench.run_plan(wl, worker, shared, False, **dev) for shared in (False, True))
    assert (p["launches"], p["short"], p["streaming"]) == (-(-wl.T // 993), 0, 0)
    passes = sum(16 + 16 * np.unique(worker[k:k + wl.K]).size for k in range(0, wl.T, wl.K))
    assert 0.5 * passes < p["bytes"] / wl.P < passes
    assert q["bytes"] < p["bytes"] / 2
    few = np.arange(wl.T, dtype=np.int32) % 5
    p = bench.run_plan(wl, few, False, False, **dev)
    assert p["bytes"] == wl.P * p["launches"] * (16 + 2 * 8 * 5)
    # adaptive staleness: half the commits a launch
    assert bench.run_plan(wl, worker, False, True, **dev)["launches"] == -(-wl.T // 495)


def test_host_description():
    d = bench.host_description()
    assert d["logical_cores"] >= 1 and (d["usable_cores"] is None or d["usable_cores"] >= 1)


def test_headline_distinct_workers_per_pass_match_schedule():
    """The bytes bench.py counts for passes come from the library; recompute D
    per pass of 32 from the schedule (host only) and compare with the per-pass
    figure recorded next to the counters."""
    import oracle as O
    from paper_1805_08469_amd.workloads import WORKLOADS
    wl = WORKLOADS["headline"]
    worker, _ = O.schedule(wl.n, wl.T, wl.law, wl.law_p0, wl.law_p1, seed=wl.seed)
    d = [np.unique(worker[k:k + wl.K]).size for k in range(0, wl.T, wl.K)]
    mean_bytes = 25_000_000 * (16 + 16 * np.mean(d))
    rec = _summary(("pass_kernel", "headline", "local"))["alg_bytes_per_launch"]
    assert rec == pytest.approx(mean_bytes, rel=0.03)
