"""CPU checks of the benchmark script's command line (no GPU needed)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_parses_and_imports():
    sys.path.insert(0, ROOT)
    import bench  # noqa: F401  (a syntax error or a broken module fails here)

    assert callable(bench.main) and callable(bench.cpu_baseline)


def test_roofline_names_the_kernel_that_was_timed():
    sys.path.insert(0, ROOT)
    import bench

    class Comp:
        def __init__(self, form):
            self.form = form

        def debug_state(self):
            return [{"form": self.form}], {}

    assert bench.timed_kernel(Comp(2)) == {"kernel": "k_dense"} and bench.timed_kernel(Comp(3)) == {"kernel": "k_dense"}
    direct = bench.timed_kernel(Comp(1))
    assert direct["kernel"] == "k_dacc" and "three later passes" in direct["not_timed"]


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
