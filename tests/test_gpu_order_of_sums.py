"""Which wave or lane holds a value must not decide the order in which it is added up: a sum's last bit does, now and then, decide a code.
Outputs of seeded networks, as digests (SHA-256, first 16 digits) of what the kernels give that the present ones took the place of."""
import hashlib

import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu

# hidden widths of 257 .. 511 (before tiles of padding were left out)
PADDED = [
    ("in sine 2x300x300x300x3", "auto", "9676dbbb4ae5e949"),
    ("in wavelet 2x400x400x400x3", "auto", "e6c9980bddc15f38"),
    ("in sine 2x449x449x449x3", "auto", "c600aabf00018985"),
    ("in complex 2x181x181x3", "auto", "3027b4153fbdd55e"),
    ("in complex 2x150x150x3", "auto", "21c2b36e33da30f9"),
]

# both sides rotated (the un-rotation as integer butterflies)
TWO_SIDED = [
    ("both sine 2x32x32x32x3", "auto", "6eb4212a6e9038e6"),
    ("both sine 2x32x32x32x3", "dyn", "03d032e767e16821"),
    ("both wavelet 2x32x32x32x3", "auto", "a76277c6d07f11e5"),
    ("both wavelet 2x32x32x32x3", "dyn", "a862b5dff340f1a2"),
    ("both sine 2x64x64x64x3", "auto", "a1b894b88fb3cbd6"),
    ("both sine 2x64x64x64x3", "dyn", "581c3bb2658b034b"),
    ("both wavelet 2x64x64x64x3", "auto", "5200c4b1c9d2a815"),
    ("both wavelet 2x64x64x64x3", "dyn", "b98db785a9a75d0a"),
    ("both sine 2x128x128x128x3", "auto", "1df235189f36de92"),
    ("both sine 2x128x128x128x3", "dyn", "3c11f1cfa807c942"),
    ("both wavelet 2x128x128x128x3", "auto", "d399539f2d5eac5d"),
    ("both wavelet 2x128x128x128x3", "dyn", "bd22c42e7395522c"),
    ("both sine 2x256x256x256x3", "auto", "036e92c9c0b17707"),
    ("both sine 2x256x256x256x3", "dyn", "140522b41dc497ba"),
    ("both wavelet 2x256x256x256x3", "auto", "b12cfc6e4a73f57e"),
    ("both wavelet 2x256x256x256x3", "dyn", "e7119cdabd6b81a2"),
]


def _points(n, k):
    """Points of [-1, 1)^k from integers alone."""
    z = (np.arange(n * k, dtype=np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
    z ^= z >> np.uint64(31)
    z *= np.uint64(0xBF58476D1CE4E5B9)
    z ^= z >> np.uint64(29)
    return ((z >> np.uint64(40)).astype(np.float64) / 2**23 - 1.0).astype(np.float32).reshape(n, k)


def _digest(network, path):
    import torch
    mode, act, shape = network.split()
    dims = [int(d) for d in shape.split("x")]
    if act == "complex":
        W, b = synth.wire_init(dims, 30.0, 7)
        m = dhq.Model.complex_wavelet(dims, 30.0, W, b, 10.0, 8, 8)
    else:
        W, b = synth.siren_init(dims, 30.0, 7)
        m = dhq.Model(dims, 30.0, W, b, 8, 8, mode={"in": dhq.DHQ_ROTATE_IN, "both": dhq.DHQ_ROTATE_BOTH}[mode],
                      wavelet_s0=10.0 if act == "wavelet" else None)
    x = torch.from_numpy(_points(20011, dims[0])).cuda()
    m.calibrate(x[::3].contiguous())
    print(f"[order of sums] {network} {path}", flush=True)
    out = m.forward(x, flags={"auto": dhq.DHQ_AUTO, "dyn": dhq.DHQ_DYNAMIC}[path]).cpu().numpy()
    m.close()
    return hashlib.sha256(out.tobytes()).hexdigest()[:16]


@pytest.mark.parametrize("network,path,digest", PADDED, ids=lambda v: v.replace(" ", "_"))
def test_padded_networks(network, path, digest):
    assert _digest(network, path) == digest


@pytest.mark.parametrize("network,path,digest", TWO_SIDED, ids=lambda v: v.replace(" ", "_"))
def test_two_sided_networks(network, path, digest):
    assert _digest(network, path) == digest
