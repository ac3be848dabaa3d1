"""Weight and bias gradients of the network against the oracle's BF16 storage model, at the
edges of their kernel: tiles shorter than 16 voxels, grids of fewer than 32 voxels, axes that
leave a tile no even split, one to four chunks of 32 input channels, one to two groups of
output channels with and without an odd last one, channel counts that are no multiple of 4
or 16, and a grid of more slices than tiles per slice."""
import numpy as np
import pytest

from oracle import unet
from gpu_util import announce, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu

# The inputs keep everything before the weight gradients exact: weights of -1, 0 and 1 (about
# three taps of an output are not 0), small whole numbers in the volumes, a scale that is a
# power of two.  Every FP32 sum of the forward pass and of the data gradients then has few
# terms on one binary grid and is exact in any order, so device and model round the same
# numbers to BF16 and hold the same activations and output gradients; what is left is the order of
# the FP32 sums over the voxels: at most about 64 dependent steps of 32 voxels and 512 slices,
# (64 + 512) 2^-24 = 3.4e-5 of the sum of magnitudes at worst and about the square root of the
# number of steps, 1.5e-6, as they fall; times 5 for cancellation.  A wrong tap, channel, voxel or
# slice gives an error near 1.
TOL = 1e-5
CASES = [
    # widths, grid, input channels
    ((4, 8), (4, 4, 4), 1),          # 2^3 voxels at the second level: less than one 32-deep step
    ((6, 10), (4, 32, 32), 3),       # 2 x 16 x 16 at the second level
    ((8, 16), (32, 8, 4), 5),        # z of 4 and 2
    ((8, 40), (8, 16, 32), 2),       # 48 input channels (two chunks), 40 outputs
    ((36, 24), (8, 8, 16), 32),      # 32 channels in, 60 of the concatenation, 36 outputs
    ((64, 48), (4, 8, 16), 7),       # four chunks, two groups with and without an odd last tile
    ((17, 48), (16, 8, 8), 30),      # one chunk of 32, strides 20 and 68
    ((4, 4), (64, 32, 64), 1),       # many slices
]


@pytest.mark.parametrize("widths,shape,in_ch", CASES)
def test_weight_gradients_vs_storage_model(widths, shape, in_ch):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("weight gradients %s %s C=%d" % (widths, shape, in_ch))
    rng = np.random.default_rng(11)
    net = mh3d.Net(widths, in_channels=in_ch, seed=0)
    lay, total = unet.param_layout(widths, in_ch)
    flat = np.zeros(total)
    for name, cin, cout, k, wo, bo in lay:
        taps = 3.0 / (cin * k ** 3)
        flat[wo:bo] = rng.choice([-1.0, 0.0, 1.0], bo - wo, p=[taps / 3, 1 - taps, 2 * taps / 3] if taps < 1 else [0.3, 0.2, 0.5])
        flat[bo:bo + cout] = rng.integers(0, 2, cout)
    net.set_params(torch.tensor(flat, dtype=torch.float32))
    x = rng.integers(-2, 3, (in_ch,) + shape).astype(np.float64)
    s = 2.0 ** np.ceil(np.log2(np.abs(x.sum(axis=0)).max()))
    x[:, 0, 0, 0] = 0.0
    x[0, 0, 0, 0] = s            # the largest |sum over the channels|
    t = rng.integers(-2, 3, shape).astype(np.float64)
    if in_ch == 1:
        x = x[0]
    xt, tt = torch.tensor(x, dtype=torch.float32), torch.tensor(t, dtype=torch.float32)
    net.loss_grad(xt, tt)
    g = net.grads().cpu().numpy()
    _, ref, _ = unet.loss_and_grads(flat, x / s, t / s, widths, bf16=True)
    err = {name: (rel_l2(g[wo:bo], ref[wo:bo]), rel_l2(g[bo:bo + cout], ref[bo:bo + cout]))
           for name, cin, cout, k, wo, bo in lay}
    print(" ".join("%s %.1e/%.1e" % (k, a, b) for k, (a, b) in err.items()), flush=True)
    assert max(max(e) for e in err.values()) <= TOL
    # a second call forms the same sums (nothing accumulates between calls)
    net.loss_grad(xt, tt)
    assert np.array_equal(net.grads().cpu().numpy(), g)
