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


class Clock:
    """Stands in for torch.cuda: an event holds the time of its last record."""
    def __init__(self):
        self.now = 0.0
        self.cuda, clock = self, self

        class Event:
            def __init__(self, enable_timing):
                self.at = None

            def record(self):
                self.at = clock.now

            def elapsed_time(self, end):
                return end.at - self.at
        self.Event = Event

    def synchronize(self):
        pass


def test_a_paired_kernel_is_timed_where_a_pass_has_one():
    """Whether a pass is one launch is what its events say: the query answers for some forms of it alone."""
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    run, clock = object.__new__(bench.LayerRun), Clock()
    run.torch, run.paired = clock, {"fwd_pair": False, "bwd_pair": False}
    launches = {0: 2.0, 1: 1.0, 2: 2.0, 3: 1.0, 4: 0.5, 6: 1.0, 7: 1.0, 8: 2.5}      # the backward pass has no paired kernel

    def step(i, profile):
        stage, begin, end = profile
        clock.now += 0.25
        if stage in launches:
            begin.record()
            clock.now += launches[stage]
            end.record()

    run.step = step
    stage_ms, kernel_ms, pair_ms = run.stage_table(reps=5)
    assert pair_ms == {"fwd_pair": 2.5} and stage_ms["fwd_Y"] == 2.0 and kernel_ms["bwd_dW"] == 0.5
