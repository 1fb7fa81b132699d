"""The two-sided network at width 512: DHQ_AUTO's whole-network kernel against the layer-by-layer kernels, bit for bit."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("dims,bits,s0", [([2, 512, 3], 8, None), ([1, 512, 512, 1], 8, None), ([3, 512, 512, 512, 32], 6, None),
                                          ([4] + [512] * 4 + [5], 4, None), ([2, 512, 512, 3], 8, 10.0), ([2, 512, 512, 17], 8, 0.0)])
def test_same_bits_as_layer_by_layer(dims, bits, s0):
    W, b = synth.siren_init(dims, 30.0, 7 + len(dims))
    m = dhq.Model(dims, 30.0, W, b, bits, bits, mode=dhq.DHQ_ROTATE_BOTH, wavelet_s0=s0)
    rng = np.random.default_rng(dims[0])
    m.calibrate(_dev(rng.uniform(-1, 1, size=(4099, dims[0])).astype(np.float32)))
    # one row, a tile less one, a tile and one, a second and a third pass of some workgroups
    for n in (1, 127, 129, 32768 + 33, 70001):
        print(f"[two-sided 512] {dims} {bits} bits s0={s0} n={n}", flush=True)
        x = _dev(rng.uniform(-1.2, 1.2, size=(n, dims[0])).astype(np.float32))
        auto, lw = _host(m.forward(x)), _host(m.forward(x, flags=dhq.DHQ_LAYERWISE))
        assert np.isfinite(lw).all() and np.abs(lw).max() > 0
        assert np.array_equal(auto, lw)
    m.close()


def test_entries_beyond_two_digits_keep_the_layer_by_layer_path():
    """A first layer with one non-zero weight: all its codes are +-127 and the un-rotated weights hold 512 * 127 > 32 639."""
    dims = [2, 512, 512, 3]
    W, b = synth.siren_init(dims, 30.0, 1)
    W[0] = np.zeros_like(W[0])
    W[0][7, 1] = 0.3
    m = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_ROTATE_BOTH)
    x = _dev(np.random.default_rng(1).uniform(-1, 1, size=(5000, 2)).astype(np.float32))
    m.calibrate(x)
    assert np.array_equal(_host(m.forward(x)), _host(m.forward(x, flags=dhq.DHQ_LAYERWISE)))
    m.close()
