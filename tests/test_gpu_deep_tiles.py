"""The deeper tiles of the default launch (several steps per launch) against one-step
launches: the same state bit for bit, since every phase runs the one-step node code on
values rounded as stored. The sizes select each of the four tile shapes, with tiles cut by
walls and by the wrap of a periodic direction (lattices narrower than a tile's ring among
them), and step counts that split into launches of every depth."""
import numpy as np
import pytest

import workloads as W
from parity import run_gpu

pytestmark = pytest.mark.gpu

WALLS = [W.dirichlet(0.5), W.robin(0.3, 1.0, -0.2)]
SIZES = [(1, 1, "periodic"), (3, 5, "periodic"), (2, 2, "walls"), (33, 7, "walls"), (17, 40, "x"), (64, 32, "y"),
         (200, 150, "walls"), (131, 190, "y"), (301, 299, "walls"), (290, 310, "x"), (520, 401, "walls"),
         (515, 430, "periodic")]


def problem(nx, ny, kind, source):
    p = [W.PERIODIC, W.PERIODIC]
    sides = {"periodic": p + p, "walls": WALLS + [W.adiabatic(0.02), W.dirichlet(0.1, -0.03)],
             "x": WALLS + p, "y": p + [W.adiabatic(), W.dirichlet(-0.4, 0.05)]}[kind]
    prob = W.problem(nx, ny, 0.04, 0.06, sides, g_beta=0.0 if "viscous" in source else 1e-4, T0=0.1, Fx=1e-5,
                     Q=2e-5, viscous_heating="viscous" in source)
    if "field" in source:
        prob["Q_field"] = W.noise_field(5, nx, ny, 1e-4).astype(np.float32)
    return prob


def fields(nx, ny):
    return {k: (W.noise_field(s, nx, ny, a)).astype(np.float32)
            for k, s, a in (("ux", 1, 0.02), ("uy", 2, 0.02), ("T", 3, 0.3))}


def state(s):
    import torch
    f, g = s.populations()
    torch.cuda.synchronize()
    return f.cpu().numpy(), g.cpu().numpy()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("source", ["", "viscous", "field", "viscous field"])
@pytest.mark.parametrize("nx,ny,kind", SIZES)
def test_default_launch_equals_single_steps(nx, ny, kind, source, precision):
    prob, f = problem(nx, ny, kind, source), fields(nx, ny)
    for steps, graph in ((1, 0), (5, 0), (13, 0), (26, 8)):
        a = state(run_gpu(prob, steps, f, precision, launch=dict(block_x=256, steps_per_launch=1)))
        b = state(run_gpu(prob, steps, f, precision, graph=graph))
        assert np.isfinite(a[0]).all()
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("nx,ny,precision", [(1010, 700, 0), (1201, 901, 1)])
def test_large_lattices_mix_launches_of_three_two_and_one(nx, ny, precision):
    prob, f = problem(nx, ny, "walls", "field"), fields(nx, ny)
    for steps, graph in ((2, 0), (3, 0), (4, 0), (6, 0), (21, 8)):
        a = state(run_gpu(prob, steps, f, precision, launch=dict(block_x=256, steps_per_launch=1)))
        b = state(run_gpu(prob, steps, f, precision, graph=graph))
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sizes", [[(33, 7), (20, 20)], [(131, 90), (64, 100), (70, 70)], [(210, 300), (130, 200)],
                                   [(520, 401), (64, 64), (300, 300)]])
def test_default_batch_equals_single_lattices(sizes, precision):
    """Batches whose node count selects each shape, with mixed source terms, through
    clbm_batch_step and through the run graph."""
    import torch
    import paper_1801_04577_amd as clbm
    sources = ["", "viscous", "field"]
    for mix in (sources[:1], sources[1:2], sources):
        probs = [problem(nx, ny, ["walls", "y", "periodic"][i % 3], mix[i % len(mix)])
                 for i, (nx, ny) in enumerate(sizes)]
        b = clbm.Batch(probs, precision=precision)
        for i, (nx, ny) in enumerate(sizes):
            b.init(i, **{k: torch.from_numpy(v) for k, v in fields(nx, ny).items()})
        b.step(7)
        b.run(max_steps=10, tol=0.0, K=10)
        for i, (nx, ny) in enumerate(sizes):
            s = run_gpu(probs[i], 17, fields(nx, ny), precision, launch=dict(block_x=256, steps_per_launch=1))
            for x, y in zip(s.macros(), b.macros(i)):
                assert torch.equal(x, y)
