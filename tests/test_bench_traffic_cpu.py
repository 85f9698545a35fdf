"""bench.py's bandwidth figures come from counted bytes: a counter summary counts
only while every source that decides what a launch moves is the one it was taken
on, and for its own form; without one no fraction of the peak is stated."""
import hashlib
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench(root, monkeypatch):
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    monkeypatch.setattr(mod, "ROOT", str(root))
    return mod


def _tree(tmp_path, form=None):
    csrc = tmp_path / "paper_2103_07537_amd" / "csrc"
    csrc.mkdir(parents=True)
    names = ("solve_kernels.hip", "solve_kernels.h", "solve_device.h", "sweep_kernels.hip", "dpp.h",
             "setup_kernels.hip", "hierarchy.hip", "memory.hip")
    for n in names:
        (csrc / n).write_text(f"// {n}\n")
    sha = hashlib.sha256("".join(f"// {n}\n" for n in names[:-1]).encode()).hexdigest()
    prof = tmp_path / "profiles"
    prof.mkdir()
    (prof / "traffic_test.txt").write_text(
        f"workload=w\nkind=0\n{'form=' + form if form else ''}\nsource_sha256={sha}\n"
        "traffic_bytes_per_launch=123\nvcycle_traffic_bytes=456\n")
    return csrc


@pytest.mark.parametrize("edited", ["solve_device.h", "sweep_kernels.hip", "setup_kernels.hip", "hierarchy.hip"])
def test_a_summary_is_dropped_with_any_source_it_depends_on(tmp_path, monkeypatch, edited):
    csrc = _tree(tmp_path)
    b = _bench(tmp_path, monkeypatch)
    assert b.measured_traffic("w", 0)[0] == 123.0
    (csrc / "memory.hip").write_text("// edited\n")   # moves nothing
    assert b.measured_traffic("w", 0)[2] == 456.0
    (csrc / edited).write_text("// edited\n")
    assert b.measured_traffic("w", 0) == (None, None, None)


def test_a_summary_is_for_its_form(tmp_path, monkeypatch):
    _tree(tmp_path, form="fp32")
    b = _bench(tmp_path, monkeypatch)
    assert b.measured_traffic("w", 0) == (None, None, None)
    assert b.measured_traffic("w", 0, "fp32")[0] == 123.0


def test_committed_summaries_state_no_more_than_the_peak():
    """Where a committed summary gives a launch's time, its counted rate stays under the peak."""
    import glob
    for path in glob.glob(os.path.join(ROOT, "profiles", "traffic_*.txt")):
        kv = dict(line.strip().split("=", 1) for line in open(path) if "=" in line and not line.startswith(" "))
        if "avg_us" in kv:
            assert float(kv["traffic_bytes_per_launch"]) / float(kv["avg_us"]) / 1e6 <= 8.0
