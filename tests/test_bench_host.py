"""Host-side checks of bench.py's contract (no GPU): one GPU only, and the counter
traffic constant is reported only for its own kernel class and sources."""
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stdout


def test_traffic_only_for_its_class_and_sources(monkeypatch):
    assert bench.measured_traffic("multidot") is None
    monkeypatch.setitem(bench.TRAFFIC, "sha256", "0" * 64)
    assert bench.measured_traffic(bench.TRAFFIC["class"]) is None


def test_jvp_bytes_count_each_face_point_once():
    """One viscous element of degree 1, by hand: 4 nodes with 4 vectors of 4 components and 8
    volume fluxes, 4 faces of 2 points with 10 terms (4 where inviscid); large viscous grids of
    degree 3 come to 232 bytes per node."""
    assert bench.jvp_bytes(1, 1, 1, True) == 8 * (4 * (16 + 8) + 8 * 10)
    assert bench.jvp_bytes(1, 1, 1, False) == 8 * (4 * (16 + 8) + 8 * 4)
    assert abs(bench.jvp_bytes(1024, 1024, 3, True) / (1024 * 1024 * 16) - 232) < 0.1
