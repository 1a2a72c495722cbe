"""Host logic of bench.py that runs without a GPU."""
import json
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120, cwd=ROOT)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


def test_traffic_is_reported_only_for_the_current_kernel_sources(tmp_path, monkeypatch):
    path = tmp_path / "traffic.json"
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(path))
    assert bench.traffic_entry("fp32", 17.5) is None                     # no summary
    path.write_text(json.dumps({"kernel_hash": bench.kernel_hash(), "fp32": {"bytes_per_launch": 123}}))
    assert bench.traffic_entry("fp32", 17.5) == 123
    assert bench.traffic_entry("fp16", 8.9) is None                      # storage not profiled
    path.write_text(json.dumps({"kernel_hash": "0" * 16, "fp32": {"bytes_per_launch": 123}}))
    assert bench.traffic_entry("fp32", 17.5) is None                     # kernel changed since


def test_timed_steps_start_at_an_even_level_after_a_call_of_their_length():
    """One-step calls leave the lattice at any level; the paired passes of the timed call need an even
    one and their workspace, which a call from an odd level of too few steps does not make."""
    class L:
        def __init__(self, at):
            self.at, self.calls = at, []

        def info(self):
            return self.at, self.at % 2, 0

        def step(self, n):
            self.calls.append(n)
            self.at += n

    for at in range(4):
        for steps in (1, 4, 5, 20, 21):
            lat = L(at)
            bench.warm_steps(lat, steps)
            assert lat.at % 2 == 0 and lat.calls[0] - at % 2 >= max(4, steps - 1), (at, steps, lat.calls)
