"""The network at grids and widths that select each convolution and weight-gradient kernel:
rows shorter and longer than the kernels' tiles and rings, rows that are and are not a
multiple of 32 pixels, images of a few pixels at the coarsest level, channel counts that
are odd multiples of 32, and both widths of the output layer. Every output and gradient
element against the reference network with BF16 storage of the operands, within the bound
derived in test_gpu_net.py (4 x 2^-8 of the element and its tensor's largest)."""
import numpy as np
import pytest

from oracle import net as ref

pytestmark = pytest.mark.gpu

CASES = [  # batch, height, width, cin, cout, widths
    (16, 16, 16, 8, 3, (32, 64, 128, 256)),
    (64, 24, 40, 8, 3, (32, 32, 64, 96)),
    (2, 64, 160, 8, 3, (32, 64, 128, 256)),
    (8, 16, 256, 3, 5, (64, 32, 96, 64)),
    (32, 32, 16, 32, 16, (96, 64, 32, 160)),
    (4, 32, 128, 9, 4, (64, 128, 64, 128)),
    (128, 40, 24, 8, 3, (96, 32, 128, 160)),
]


def worst(got, want):
    """Largest deviation in units of 2^-8 (|want| + max |want|)."""
    return float((np.abs(got - want) / np.maximum(2.0 ** -8 * (np.abs(want) + np.abs(want).max()), 1e-300)).max())


@pytest.mark.parametrize("B,H,W,cin,cout,widths", CASES)
def test_shapes_elementwise(B, H, W, cin, cout, widths):
    import torch
    import paper_1801_04577_amd as clbm
    rng = np.random.default_rng(B + H + W)
    params = [(w.astype(np.float32).astype(np.float64),
               rng.normal(scale=0.05, size=b.shape).astype(np.float32).astype(np.float64))
              for w, b in ref.init_params(cin, cout, widths, seed=3)]
    xs = rng.normal(size=(B, cin, H, W)).astype(np.float32)
    ts = rng.normal(scale=0.5, size=(B, cout, H, W)).astype(np.float32)
    n = clbm.Net(B, H, W, cin, cout, widths)
    n.set_params(torch.from_numpy(np.concatenate([np.concatenate([w.reshape(-1), b]) for w, b in params])
                                  .astype(np.float32)))
    y = n.forward(torch.from_numpy(xs)).cpu().numpy().astype(np.float64)
    loss = n.backward(torch.from_numpy(ts))
    grads = n.grads().cpu().numpy().astype(np.float64)
    want_y = np.stack([ref.forward(params, x.astype(np.float64), quant=True) for x in xs])
    want_loss, want = ref.loss_and_grads(params, xs.astype(np.float64), ts.astype(np.float64), quant=True)
    ratios, k = [worst(y, want_y)], 0
    for ww, wb in want:
        for t in (ww, wb):
            ratios.append(worst(grads[k:k + t.size].reshape(t.shape), t))
            k += t.size
    print("worst %.3f of the unit" % max(ratios), flush=True)
    assert loss == pytest.approx(want_loss, rel=1e-3)
    assert max(ratios) <= 4.0


@pytest.mark.parametrize("sh,sw,dh,dw,nf", [(5, 7, 3, 4, 1), (16, 12, 33, 20, 3), (9, 9, 21, 30, 2), (128, 64, 96, 7, 16)])
def test_resample_widths(sh, sw, dh, dw, nf):
    """Rows that are and are not a multiple of four cells, against 64 bits. A coordinate is off by
    at most four roundings of its size, which moves a value by at most twice the fields' largest
    times that; the sum of four products and the affine map add eight roundings."""
    import torch
    import paper_1801_04577_amd as clbm
    src = np.random.default_rng(dw).normal(size=(nf, sh, sw)).astype(np.float32)
    scale, shift = [1.0 + 0.5 * f for f in range(nf)], [0.25 * f for f in range(nf)]
    got = clbm.resample(torch.from_numpy(src).cuda(), dh, dw, scale=scale, shift=shift).cpu().numpy().astype(np.float64)

    def axis(n, m):
        f = np.clip((np.arange(m) + 0.5) * n / m - 0.5, 0, n - 1)
        lo = f.astype(int)
        return lo, np.minimum(lo + 1, n - 1), f - lo
    y0, y1, ty = axis(sh, dh)
    x0, x1, tx = axis(sw, dw)
    s = src.astype(np.float64)
    rows = s[:, y0] * (1 - ty)[None, :, None] + s[:, y1] * ty[None, :, None]
    want = rows[:, :, x0] * (1 - tx) + rows[:, :, x1] * tx
    want = want * np.array(scale)[:, None, None] + np.array(shift)[:, None, None]
    big = np.abs(s).max() * max(scale) + max(shift)
    assert np.abs(got - want).max() <= 2.0 ** -24 * (8 + 8 * (sh + sw)) * big


# What the cases above do not reach: eight rows per wave (images and batches that give every SIMD two
# waves) with each epilogue, tiles of two waves by two channel groups and those over 64 KB of LDS, layers
# whose tile does not fit in LDS at all (more than 455 input channels, four blocks of pixels per wave),
# the output layer from 32 channels to more than four and from 480, rings of 512 pixels and rings
# per kernel row where rows are no multiple of 32.
LARGE_CASES = [
    (32, 64, 64, 8, 3, (64, 128, 32, 32)),
    (16, 64, 64, 8, 3, (128, 64, 32, 32)),
    (512, 16, 16, 8, 3, (64, 32, 32, 32)),
    (48, 64, 64, 8, 3, (32, 192, 32, 32)),
    (16, 96, 80, 8, 5, (32, 64, 128, 256)),
    (16, 16, 176, 8, 3, (32, 128, 32, 32)),
    (16, 16, 208, 3, 4, (64, 32, 32, 32)),
    (32, 16, 24, 4, 4, (480, 32, 32, 32)),
]


@pytest.mark.parametrize("B,H,W,cin,cout,widths", LARGE_CASES)
def test_large_shapes_elementwise(B, H, W, cin, cout, widths):
    test_shapes_elementwise(B, H, W, cin, cout, widths)


@pytest.mark.parametrize("cout", [4, 5])
def test_output_layer_from_many_channels(cout):
    """480 channels to the output, whose tile does not fit in LDS. The outputs only, in the same unit:
    64 pixels of 32 channels at the coarsest level are too few for the gradients' bound (the reference
    with BF16 storage lies 15 units from the one without there, and the gradients 10 from either)."""
    import torch
    import paper_1801_04577_amd as clbm
    B, H, W, cin, widths = 16, 16, 16, 4, (480, 32, 32, 32)
    rng = np.random.default_rng(cout)
    params = [(w.astype(np.float32).astype(np.float64),
               rng.normal(scale=0.05, size=b.shape).astype(np.float32).astype(np.float64))
              for w, b in ref.init_params(cin, cout, widths, seed=3)]
    xs = rng.normal(size=(B, cin, H, W)).astype(np.float32)
    n = clbm.Net(B, H, W, cin, cout, widths)
    n.set_params(torch.from_numpy(np.concatenate([np.concatenate([w.reshape(-1), b]) for w, b in params])
                                  .astype(np.float32)))
    y = n.forward(torch.from_numpy(xs)).cpu().numpy().astype(np.float64)
    want = np.stack([ref.forward(params, x.astype(np.float64), quant=True) for x in xs])
    assert worst(y, want) <= 4.0
