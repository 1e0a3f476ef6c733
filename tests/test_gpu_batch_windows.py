"""The tiles that the library picks for a batch against its two-step launches over the same
lattices, in time: a kernel variant that loses a workgroup per CU, or tiles that do not pay
over a short window, give the right states and are seen by nothing else. The two are timed in
turn; each side's best of a few runs varies by less than 2 %, and a variant that spilled or
lost half of its waves took 13 to 50 % longer."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# 64 x 14 tiles with two steps per launch, one workgroup per tile
TWO_STEP = dict(tile_x=64, tile_y=14, steps_per_launch=2, persistent_wgs=1 << 30)
SLACK = 1.08


def batch(sizes, sources, precision, launch):
    import numpy as np
    import torch
    import paper_1801_04577_amd as clbm
    walls = [W.dirichlet(0.5), W.dirichlet(-0.5), W.adiabatic(), W.adiabatic()]
    probs = []
    for i, (nx, ny) in enumerate(sizes):
        src = sources[i % len(sources)]
        p = W.problem(nx, ny, 0.04, 0.06, walls, g_beta=0.0 if src == "viscous" else 1e-5, Q=1e-6,
                      viscous_heating=src == "viscous")
        if src == "field":
            p["Q_field"] = np.full((ny, nx), 1e-6, np.float32)
        probs.append(p)
    b = clbm.Batch(probs, launch=launch, precision=precision)
    for i, (nx, ny) in enumerate(sizes):
        b.init(i, T=torch.from_numpy(W.noise_field(i, nx, ny, 1e-3).astype(np.float32)))
    return b


def per_call(call, calls):
    import torch
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(calls):
        call()
    end.record()
    end.synchronize()
    return start.elapsed_time(end) / calls


def assert_no_slower(sizes, sources, precision, call, calls):
    own, two = batch(sizes, sources, precision, None), batch(sizes, sources, precision, TWO_STEP)
    best = [1e9, 1e9]
    for attempt in range(10):
        for k, b in enumerate((own, two)):
            best[k] = min(best[k], per_call(lambda: call(b), calls))
        if attempt >= 3 and best[0] <= SLACK * best[1]:
            break
    print("%.1f us a call, two-step launches %.1f us" % (1e3 * best[0], 1e3 * best[1]), flush=True)
    assert best[0] <= SLACK * best[1]


@pytest.mark.parametrize("sizes", [[(330, 330)] * 8, [(512, 512)] * 16, [(64 + 7 * i, 64 + 7 * i) for i in range(64)]])
def test_mixed_sources(sizes):
    assert_no_slower(sizes, ["", "viscous", "field"], 0, lambda b: b.step(20), 10)


@pytest.mark.parametrize("sizes,precision,call", [
    ([(300, 300)] * 4, 1, lambda b: b.step(1)), ([(300, 300)] * 4, 1, lambda b: b.step(2)),
    ([(330, 330)] * 8, 1, lambda b: b.step(2)), ([(330, 330)] * 8, 1, lambda b: b.step(4)),
    ([(512, 512)] * 16, 0, lambda b: b.step(2)), ([(64 + 4 * i, 60 + 3 * i) for i in range(24)], 1, lambda b: b.step(2)),
    ([(512, 512)] * 16, 0, lambda b: b.run(40, 0.0, K=2))])
def test_short_windows(sizes, precision, call):
    assert_no_slower(sizes, [""], precision, call, 40)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sizes", [[(64, 2), (40, 3)], [(300, 300)] * 4, [(700, 640)] * 3])
def test_short_windows_keep_the_state(sizes, precision):
    """Calls that mix deeper launches with pairs and lone steps over the second tile list, and
    lists too small for it, against two-step launches: the same bits."""
    import torch
    sources = ["", "viscous", "field"]
    own, two = batch(sizes, sources, precision, None), batch(sizes, sources, precision, TWO_STEP)
    for n in (1, 2, 4, 7, 8, 1, 3, 5):
        own.step(n)
        two.step(n)
        for i in range(own.n):
            for x, y in zip(own.macros(i), two.macros(i)):
                assert torch.equal(x, y), (n, i)
