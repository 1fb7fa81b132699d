"""fp32-activation networks: the whole-network kernel against the layer-by-layer kernels, and weights and activations of every size."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from oracle import dhq_oracle as o
from paper_2508_13478_amd import synth
from test_gpu_variants import FLOAT_TOL_WIDE

pytestmark = pytest.mark.gpu

# widths on both sides of every tile shape's range, unequal ones, fan-ins beyond a k block, outputs beyond a tile, one hidden layer
SHAPES = [[1, 1, 1], [2, 32, 32, 3], [4, 33, 33, 5], [2, 64, 64, 3], [3, 65, 128, 2], [40, 48, 17, 64, 100], [2, 129, 200, 1], [2, 256, 256, 3],
          [17, 257, 64, 33], [2, 100, 500, 40, 3], [2, 512, 512, 3],
          # both sides of the rule that sends large fan-ins, fan-outs and widths layer by layer
          [300, 30, 3], [200, 60, 60, 2], [65, 256, 256, 3], [2, 128, 128, 70], [2, 40, 40, 40], [3, 384, 416, 2],
          [2, 300, 300, 300, 3], [40, 352, 352, 352, 32], [64, 257, 3], [64, 128, 3], [17, 64, 3]]


@pytest.mark.parametrize("dims", SHAPES, ids=["x".join(map(str, d)) for d in SHAPES])
@pytest.mark.parametrize("s0", [None, 10.0], ids=["sine", "wavelet"])
def test_same_bits_as_layer_by_layer(dims, s0):
    """The same pieces, products and order of sums, so the same bits, whatever the tile: one row, the edges of a tile, of one round of
    the small tiles on 256 CUs, and several rounds with a ragged end."""
    import torch
    W, b = synth.siren_init(dims, 30.0, 77 + sum(dims))
    m = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32, wavelet_s0=s0)
    g = torch.Generator(device="cuda").manual_seed(9)
    for n in (1, 32, 33, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16385, 32769, 49153, 65537, 140001):
        print(f"[float net] {dims} s0={s0} n={n}", flush=True)
        x = torch.rand((n, dims[0]), generator=g, device="cuda") * 2 - 1
        assert torch.equal(m.forward(x), m.forward(x, flags=dhq.DHQ_LAYERWISE))
    m.close()


@pytest.mark.parametrize("width", [32, 48, 256])
def test_weights_of_very_different_sizes(width):
    """A feature that is zero for every coordinate, with weights 2^40 times the others': the others keep fp32 accuracy."""
    dims = [2, width, width, 3]
    W, b = synth.siren_init(dims, 30.0, 5)
    W[0][0], b[0][0] = 0.0, 0.0
    for l in (1, 2):
        W[l][:, 0] = 2.0 ** 40
    W[1][0, :], b[1][0] = 0.0, 0.0
    x = synth.grid_coords(40)
    import torch
    m = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32)
    exp, _ = o.mlp_float(dims, 30.0, W, b, x)
    for flags in (dhq.DHQ_AUTO, dhq.DHQ_LAYERWISE):
        out = m.forward(torch.from_numpy(x).to("cuda"), flags=flags)
        err = np.abs(out.cpu().numpy().astype(np.float64) - exp).max()
        print(f"[float net] width {width} flags {flags}: max-abs err {err:.2e}", flush=True)
        assert err <= FLOAT_TOL_WIDE
    m.close()


@pytest.mark.parametrize("scale", [1e-4, 1e-8, 1e-10])
@pytest.mark.parametrize("width", [32, 48, 128, 256, 300, 512])
@pytest.mark.parametrize("s0", [None, 10.0], ids=["sine", "wavelet"])
def test_small_activations(s0, width, scale):
    """A first layer whose activations are all of the size of `scale` (small arguments; the tail of the wavelet's envelope), a second one
    whose weights bring them back: fp32 accuracy does not depend on a value's size.  The second layer's arguments, up to about 100
    radians, are rounded to 2^-24 of themselves, 6e-6, which the output layer's weights (sqrt(6 / K) / 30, K of them with random
    signs) take to 5e-7, and a few such roundings to a few times that; a scale that a layer shares leaves 1e-4 and more."""
    import torch
    dims = [2, width, width, 3]
    W, b = synth.siren_init(dims, 30.0, 5)
    if s0 is None:
        W[0], b[0] = (W[0] * np.float32(scale)).astype(np.float32), (b[0] * np.float32(scale)).astype(np.float32)
    else:
        W[0] = (W[0] * np.float32(1e-3)).astype(np.float32)
        b[0][:] = np.sqrt(-np.log(scale)) / s0
    W[1] = (W[1] / np.float32(scale)).astype(np.float32)
    x = synth.grid_coords(30)
    exp, _ = o.mlp_float(dims, 30.0, W, b, x, **({"gabor_s0": s0} if s0 is not None else {}))
    m = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32, wavelet_s0=s0)
    for flags in (dhq.DHQ_AUTO, dhq.DHQ_LAYERWISE):
        err = np.abs(m.forward(torch.from_numpy(x).to("cuda"), flags=flags).cpu().numpy().astype(np.float64) - exp).max()
        print(f"[float net] width {width} s0={s0} scale {scale} flags {flags}: max-abs err {err:.2e}", flush=True)
        assert err <= FLOAT_TOL_WIDE
    m.close()


@pytest.mark.parametrize("width", [32, 48, 128, 256, 300])
@pytest.mark.parametrize("s0", [None, 0.1], ids=["sine", "wavelet"])
def test_coordinates_beyond_the_largest_bf16(s0, width):
    """Coordinates of 3.39e38 to 3.40e38, of which the first bf16 piece would round to infinity, with weights that are powers of two (their
    own first piece): arguments of up to 24."""
    import torch
    dims = [2, width, width, 3]
    W, b = synth.siren_init(dims, 30.0, 5)
    rng = np.random.default_rng(width)
    W[0] = (rng.choice([-1.0, 1.0], W[0].shape) * np.exp2(rng.choice([-126.0, -125.0], W[0].shape))).astype(np.float32)
    x = (rng.choice([-1.0, 1.0], (700, 2)) * rng.uniform(3.38e38, 3.4028e38, (700, 2))).astype(np.float32)
    exp, _ = o.mlp_float(dims, 1.0, W, b, x, **({"gabor_s0": s0} if s0 is not None else {}))
    m = dhq.Model(dims, 1.0, W, b, mode=dhq.DHQ_W32A32, wavelet_s0=s0)
    for flags in (dhq.DHQ_AUTO, dhq.DHQ_LAYERWISE):
        err = np.abs(m.forward(torch.from_numpy(x).to("cuda"), flags=flags).cpu().numpy().astype(np.float64) - exp).max()
        print(f"[float net] width {width} s0={s0} flags {flags}: max-abs err {err:.2e}", flush=True)
        assert err <= FLOAT_TOL_WIDE
    m.close()
