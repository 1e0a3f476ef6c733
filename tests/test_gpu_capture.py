"""Steps recorded into a caller's stream capture and replayed: the recorded launches go from the
buffer that held the state to the one that holds it afterwards, so they can be repeated where
that is the same one. It is for every multiple of four steps, as with two-step launches."""
import pytest

import workloads as W
from parity import f32

pytestmark = pytest.mark.gpu

REPLAYS = 3


def noise(prob, seed):
    import torch
    return torch.from_numpy(f32(prob["T0"] + W.noise_field(seed, prob["nx"], prob["ny"], 1e-3)))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny", [(64, 32), (200, 150), (390, 380), (520, 400), (1010, 700)])
def test_captured_steps_of_a_lattice(nx, ny, precision):
    import torch
    import paper_1801_04577_amd as clbm
    prob, stream = W.cavity(nx, ny, Ra=1e4, Pr=0.71), torch.cuda.Stream()
    for n in (3, 4, 7, 8, 16, 20, 28, 100):
        with torch.cuda.stream(stream):
            s, alone = clbm.Solver(prob, precision, stream=stream), clbm.Solver(prob, precision, stream=stream)
            for v in (s, alone):
                v.init(T=noise(prob, n))
                v.step(4)
            stream.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                s.step(n)
            for k in range(REPLAYS):
                g.replay()
                alone.step(n)
                for x, y in zip(s.macros(), alone.macros()):
                    assert torch.equal(x, y), (n, k)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sizes", [[(33, 17), (20, 20)], [(131, 90), (64, 100), (70, 70)], [(520, 401), (64, 64), (300, 300)]])
def test_captured_steps_of_a_batch(sizes, precision):
    import torch
    import paper_1801_04577_amd as clbm
    probs, stream = [W.cavity(nx, ny, Ra=1e4, Pr=0.71) for nx, ny in sizes], torch.cuda.Stream()
    for n in (3, 4, 7, 8, 16, 20, 28, 100):
        with torch.cuda.stream(stream):
            b = clbm.Batch(probs, precision=precision, stream=stream)
            alone = [clbm.Solver(p, precision, stream=stream) for p in probs]
            for i, p in enumerate(probs):
                b.init(i, T=noise(p, n + i))
                alone[i].init(T=noise(p, n + i))
            b.step(4)
            stream.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                b.step(n)
            for k in range(REPLAYS):
                g.replay()
                for i, s in enumerate(alone):
                    s.step(n if k else n + 4)
                    for x, y in zip(b.macros(i), s.macros()):
                        assert torch.equal(x, y), (n, k, i)
