"""bench.py's command line on the CPU: it measures one GPU and refuses a
multi-GPU request before touching any device."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 2
    assert "one GPU only" in r.stderr and r.stdout == ""


def test_counter_traffic_belongs_to_the_kernels_that_ran(monkeypatch, tmp_path):
    """Counted bytes are reported only for the same sources and steps per pass; the
    sources include the rules that choose the kernels."""
    import json

    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    from paper_1511_04633_amd import profiling

    assert "csrc/host.hpp" in profiling.KERNEL_SOURCES
    os.makedirs(tmp_path / "profiles")
    entry = {"traffic_bytes": 1, "steps_per_pass": 2, "source_sha256": profiling.kernel_source_hash()}
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps({"f32_256": entry}))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.counter_traffic("f32", 256, 2) == entry
    assert bench.counter_traffic("f32", 256, 1) is None
    assert bench.counter_traffic("f64", 256, 2) is None
    entry["source_sha256"] = "0"
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps({"f32_256": entry}))
    assert bench.counter_traffic("f32", 256, 2) is None
