"""bench.py accounts for the launches that the library makes: a lattice that runs several steps per
launch on the library's own tiles has no two-step launches to report a bandwidth of, whichever way the
launch shape was given."""
import json
import os
import subprocess
import sys

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("launch,kernel", [(None, None), ("256,1,1,1,2", None), ("256,1,1,1,2,14", "k_step2"),
                                           ("256,1,1,1,1", "k_step")])
def test_roofline_of_a_small_lattice(launch, kernel):
    cmd = [sys.executable, "bench.py", "--n", "512", "--steps", "20", "--warmup", "4", "--no-cpu-baseline"]
    r = subprocess.run(cmd + (["--launch", launch] if launch else []), capture_output=True, text=True, timeout=100,
                       cwd=ROOT)
    assert r.returncode == 0, r.stderr
    out = json.loads(r.stdout.strip().splitlines()[-1])
    assert out["value"] > 0
    if kernel is None:
        assert out["roofline"] is None and "up to three steps per launch" in out["config"]["workload"]
        assert "per launch of 2 step(s)" not in r.stderr
    else:
        assert out["roofline"]["kernel"] == kernel


@pytest.mark.parametrize("nx,ny,precision,steps", [(64, 32, 0, 6), (256, 256, 0, 6), (384, 384, 0, 4), (512, 512, 1, 3),
                                                   (2000, 1000, 1, 2)])
def test_steps_per_launch(nx, ny, precision, steps):
    import paper_1801_04577_amd as clbm
    s = clbm.Solver(W.cavity(nx, ny), precision)
    assert s.steps_per_launch() == steps
    s.set_launch(256, 1, 1, 1, 2, 14)
    assert s.steps_per_launch() == 2
    s.set_launch(256, 1, 1, 1, 1)
    assert s.steps_per_launch() == 1
