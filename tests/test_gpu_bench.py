"""bench.py on the GPU: its JSON line for the tiny workload under each option
(one call a step or one a pass, histogram recording, a forced cache policy, the
segment scope, the shared moment), one timed step each, and for the small
workload, whose runs the run kernel takes."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = [
    ("tiny", [], "short_run_kernel<Fast>"),
    ("tiny", ["--proxy", "global", "--cache", "keep"], "short_run_kernel<FastGlobal>"),
    ("small", [], "run_kernel<Fast>"),
    ("small", ["--cache", "stream", "--kappa", "2"], "run_kernel<General, streaming>"),
    ("tiny", ["--pi-hist"], "pass_kernel<Generated, Fast, recording, depth 2>"),
    ("tiny", ["--pi-hist", "--proxy", "global"], "pass_kernel<Generated, FastGlobal, diagnostic, depth 2>"),
    ("tiny", ["--calls", "pass", "--cache", "stream"], "pass_kernel<Generated, Fast, depth 1, streaming>"),
    ("tiny", ["--calls", "pass", "--proxy", "global", "--cache", "keep"],
     "pass_kernel<Generated, FastGlobal, depth 1>"),
    ("tiny", ["--pi-scope", "segment"], "seg_step_kernel + seg_blocks_kernel"),
]


@pytest.mark.parametrize("workload,extra,label", CASES, ids=[" ".join([c[0], *c[1]]) for c in CASES])
def test_bench_line(workload, extra, label):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cmd = [sys.executable, "-u", os.path.join(ROOT, "bench.py"), "--workload", workload,
           "--steps", "1", "--warmup", "0", "--no-cpu-baseline", *extra]
    print("[bench]", workload, " ".join(extra), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    d = json.loads(r.stdout.strip().splitlines()[-1])
    assert d["value"] > 0 and d["n_gpus"] == 1 and d["steps"] == 1
    roof = d["roofline"]
    assert roof["kernel"] == label
    if workload == "tiny" or "--cache" in extra:     # no counters for these
        assert roof["traffic"] is None
    assert roof["avg_launch_ms"] * roof["launches_per_step"] == pytest.approx(d["ms_per_step"])
    if roof["bound"] == "hbm":
        assert 0 < roof["frac"] < 1
    else:   # against the VALU ceiling; the instruction count needs counters
        assert roof["bound"] == "alu" and 0 < roof["frac_of_compute_floor"] <= 1.2
        assert roof["frac"] is None or 0 < roof["frac"] < 1
