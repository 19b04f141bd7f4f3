"""Host logic of bench.py that needs no GPU."""
import importlib.util
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert p.returncode == 2
    assert "single-GPU" in p.stderr and p.stdout.strip() == ""


def test_counter_figures_of_other_kernels_are_not_reported(tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    csrc, profiles = tmp_path / "paper_2201_13195_amd" / "csrc", tmp_path / "profiles"
    csrc.mkdir(parents=True)
    profiles.mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (csrc / "a.hip").write_text("int f() { return 1; }  // one\n")
    (profiles / "hbm_traffic.txt").write_text("kernels_digest %s\ntraffic_bytes_per_launch w s 12\n" % bench.kernels_digest())
    assert bench.read_traffic("w", "s", bench.kernels_digest()) == 12.0 and bench.read_traffic("w", "t", bench.kernels_digest()) is None
    (csrc / "a.hip").write_text("// another comment\nint f() {\n    return 1;\n}\n")
    assert bench.read_traffic("w", "s", bench.kernels_digest()) == 12.0
    (csrc / "a.hip").write_text("int f() { return 2; }\n")
    assert bench.read_traffic("w", "s", bench.kernels_digest()) is None
