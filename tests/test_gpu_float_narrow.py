"""fp32-activation networks whose layers are at most 64 wide, layer by layer: one wave per tile with the layer's weights in registers."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from oracle import dhq_oracle as o
from paper_2508_13478_amd import synth
from test_gpu_variants import FLOAT_TOL_WIDE

pytestmark = pytest.mark.gpu


def _tol(dims):
    """The bounds of the wider networks' tests: sums of fp32 accuracy ahead of the hardware sine, which many inputs to the first layer
    take further into its range."""
    return FLOAT_TOL_WIDE if dims[0] <= 8 else 5e-5

SHAPES = [[2, 20, 20, 3], [1, 1, 1], [3, 32, 32, 32, 1], [4, 33, 33, 5], [2, 64, 64, 64, 3], [40, 48, 17, 64, 100], [64, 31, 2], [5, 7], [64, 512],
          [17, 64, 32, 33]]


def _rows(dims, n, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((n, dims[0]), generator=g, device="cuda") * 2 - 1


@pytest.mark.parametrize("dims", SHAPES, ids=["x".join(map(str, d)) for d in SHAPES])
@pytest.mark.parametrize("s0", [None, 10.0], ids=["sine", "wavelet"])
def test_narrow_against_oracle_and_the_wide_kernels(dims, s0):
    """Against the oracle, and (sines bit for bit) against the same network on the kernels of the wider ones: embedded in hidden widths of
    80, whose further features have no weights in or out and add nothing but zeros to any sum.  (A single layer has no hidden
    width to embed; its fan-in is embedded in 80.)"""
    import torch
    L = len(dims) - 1
    W, b = synth.siren_init(dims, 30.0, 900 + sum(dims))
    wide = [dims[0]] + [80] * (L - 1) + [dims[-1]] if L > 1 else [80, dims[-1]]
    We, be = [], []
    for l in range(L):
        w = np.zeros((wide[l + 1], wide[l]), np.float32)
        w[:dims[l + 1], :dims[l]] = W[l]
        v = np.zeros(wide[l + 1], np.float32)
        v[:dims[l + 1]] = b[l]
        We.append(w), be.append(v)
    m = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32, wavelet_s0=s0)
    mw = dhq.Model(wide, 30.0, We, be, mode=dhq.DHQ_W32A32, wavelet_s0=s0)
    # one row, a tile's edges, more tiles than waves, more than one chunk of rows
    for n in (1, 31, 33, 4097, 131072 + 77, 300001):
        if n > 5000 and dims[-1] > 64:
            continue
        print(f"[float narrow] {dims} s0={s0} n={n}", flush=True)
        x = _rows(dims, n, n)
        out = m.forward(x, flags=dhq.DHQ_LAYERWISE)
        xe = torch.zeros((n, wide[0]), device="cuda")
        xe[:, :dims[0]] = x
        ref = mw.forward(xe, flags=dhq.DHQ_LAYERWISE)
        # (wavelets bit for bit: test_narrow_wavelets_are_the_wide_kernels)
        assert torch.equal(out, ref) if s0 is None or L == 1 else float((out - ref).abs().max()) <= _tol(dims)
        idx = np.unique(np.concatenate([np.arange(min(n, 70)), np.arange(max(0, n - 70), n)]))
        exp, _ = o.mlp_float(dims, 30.0, W, b, x.cpu().numpy()[idx], **({"gabor_s0": s0} if s0 is not None else {}))
        err = np.abs(out.cpu().numpy()[idx].astype(np.float64) - exp).max()
        print(f"  max-abs err {err:.2e}", flush=True)
        assert err <= _tol(dims) * max(1.0, np.abs(exp).max())
    m.close()
    mw.close()


@pytest.mark.parametrize("dims", [d for d in SHAPES if len(d) > 2], ids=lambda d: "x".join(map(str, d)))
def test_narrow_wavelets_are_the_wide_kernels(dims):
    """Bit for bit, in the same embedding: what both split into pieces is the wavelet rounded to fp32."""
    import torch
    L = len(dims) - 1
    W, b = synth.siren_init(dims, 30.0, 900 + sum(dims))
    wide = [dims[0]] + [80] * (L - 1) + [dims[-1]]
    We = [np.pad(W[l], ((0, wide[l + 1] - dims[l + 1]), (0, wide[l] - dims[l]))) for l in range(L)]
    be = [np.pad(b[l], (0, wide[l + 1] - dims[l + 1])) for l in range(L)]
    m, mw = (dhq.Model(d, 30.0, w, v, mode=dhq.DHQ_W32A32, wavelet_s0=10.0) for d, w, v in ((dims, W, b), (wide, We, be)))
    for n in (1, 33, 4097):
        print(f"[float narrow] {dims} wavelet n={n}", flush=True)
        x = _rows(dims, n, n)
        assert torch.equal(m.forward(x, flags=dhq.DHQ_LAYERWISE), mw.forward(x, flags=dhq.DHQ_LAYERWISE))
    m.close()
    mw.close()


@pytest.mark.parametrize("dims,most", [([2, 32, 32, 3], 17), ([2, 64, 64, 3], 34), ([2, 128, 128, 3], 101), ([2, 20, 20, 3], 68),
                                       ([2, 48, 48, 48, 3], 68), ([2, 300, 300, 3], 202)])
def test_workspace_of_a_model(dims, most):
    """Device memory that a model holds, in MB: 65 536 rows of the layer-by-layer path's two buffers where DHQ_AUTO is the
    whole-network kernel, 64 MiB in narrow networks, 192 MiB in wide ones (and a little for weights and the allocator's rounding)."""
    import torch
    W, b = synth.siren_init(dims, 30.0, 1)
    first = dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32)  # the library's own image is loaded now
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    models = [dhq.Model(dims, 30.0, W, b, mode=dhq.DHQ_W32A32) for _ in range(4)]
    used = (free - torch.cuda.mem_get_info()[0]) / 4e6
    print(f"[float workspace] {dims}: {used:.1f} MB a model", flush=True)
    assert used <= most + 5
    for m in models + [first]:
        m.close()
