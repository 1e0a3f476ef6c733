"""The run graph of a batch after steps outside it. Launches take the populations from one of
two buffers to the other, so a graph belongs to the buffer that it was built for: a run
with the same arguments may find the state in the other one."""
import pytest

import workloads as W
from parity import f32

pytestmark = pytest.mark.gpu

# sizes that select each tile shape of the default launch
SIZES = [[(33, 7), (20, 20)], [(131, 90), (64, 100), (70, 70)], [(210, 300), (130, 200)],
         [(520, 401), (64, 64), (300, 300)]]
LAUNCHES = [None, dict(tile_x=128, tile_y=2), dict(tile_x=64, tile_y=14, steps_per_launch=2, persistent_wgs=40)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("launch", LAUNCHES)
@pytest.mark.parametrize("sizes", SIZES)
def test_run_after_steps_outside_the_graph(sizes, launch, precision):
    """After each kind of interruption the batch is where its lattices are when they advance
    alone, bit for bit: with the state of the run before, and with fields set in between."""
    import torch
    import paper_1801_04577_amd as clbm
    probs = [W.cavity(nx, ny, Ra=1e4 * (i + 1), Pr=0.71) for i, (nx, ny) in enumerate(sizes)]

    def fields(seed):
        return [torch.from_numpy(f32(p["T0"] + W.noise_field(seed + i, p["nx"], p["ny"], 1e-3)))
                for i, p in enumerate(probs)]

    b = clbm.Batch(probs, launch=launch, precision=precision)
    singles = [clbm.Solver(p, precision) for p in probs]

    def init(seed):
        for i, T in enumerate(fields(seed)):
            b.init(i, T=T)
            singles[i].init(T=T)

    def run():
        steps, status = b.run(12, 0.0, K=6)
        assert steps == [12] * b.n and set(status) == {"max_steps"}
        for s in singles:
            s.step(12)

    def check(what):
        for i, s in enumerate(singles):
            for x, y in zip(b.macros(i), s.macros()):
                assert torch.equal(x, y), (what, i)

    init(1)
    run()
    check("first run")
    for n in (1, 4, 3, 100):   # one step is one launch, whatever the tiles
        b.step(n)
        for s in singles:
            s.step(n)
        run()
        check("run after step(%d)" % n)
        b.step(n)
        init(10 * n)
        run()
        check("run after step(%d) and init" % n)
