"""bench.py command line on the CPU: a request for more than one GPU is refused with a JSON error line
and exit status 2, before anything touches a GPU."""

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 2
    line = json.loads(r.stdout.strip().splitlines()[-1])
    assert line["n_gpus"] == 2 and "one GPU" in line["error"]


def test_the_shape_that_bench_reports_is_the_one_it_set():
    """Without the autotuner the headline leg reports a shape that the simulation was given."""
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench

    class Sim:
        def __init__(self):
            self.calls = []

        def set_kernel_config(self, *shape):
            self.calls.append(shape)

    for kernel in (None, "1,8,32", "4,4,64,2"):
        sim = Sim()
        shape, tune = bench.choose_shape(sim, kernel, False)
        assert sim.calls == [shape] and tune is None
        assert kernel is None or shape == tuple(int(v) for v in kernel.split(","))
