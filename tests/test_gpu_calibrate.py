"""Calibration on the per-layer kernels of the fused networks: the layer-by-layer path's scales, bit for bit."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu


def _scales(m, x):
    m.calibrate(x)
    got = m.scales()[1].copy()
    m.forward(x, flags=dhq.DHQ_LAYERWISE | dhq.DHQ_DYNAMIC)
    return got, m.dynamic_scales()


@pytest.mark.parametrize("dims", [[2, 32, 3], [1, 32, 32, 32, 1], [3, 64, 64, 2], [2, 128, 128, 128, 3], [4, 256, 256, 256, 5], [2, 20, 20, 3],
                                  [3, 90, 120, 1], [2, 150, 150, 3], [1, 180, 180, 180, 2], [2, 200, 200, 200, 3]], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("act,bits", [("sine", 8), ("sine", 4), ("wavelet", 8), ("complex", 8)])
def test_scales_of_every_activation_and_width(dims, act, bits):
    """Every tile count of the transform (its stage over the lane halves differs below four tiles), rows at the edges of a wave's and
    a workgroup's tile, and several passes."""
    import torch
    if act == "complex":
        dims = [dims[0]] + [max(1, d // 2) for d in dims[1:-1]] + [dims[-1]]
        W, b = synth.wire_init(dims, 30.0, 3)
        m = dhq.Model.complex_wavelet(dims, 30.0, W, b, 10.0, bits, bits)
    else:
        W, b = synth.siren_init(dims, 30.0, 3)
        m = dhq.Model(dims, 30.0, W, b, bits, bits, wavelet_s0=10.0 if act == "wavelet" else None)
    g = torch.Generator(device="cuda").manual_seed(4)
    for n in (1, 33, 257, 70001):
        print(f"[calibrate] {dims} {act} {bits} bits n={n}", flush=True)
        x = torch.rand((n, dims[0]), generator=g, device="cuda") * 2 - 1
        got, exp = _scales(m, x)
        assert np.array_equal(got, exp)
    m.close()


@pytest.mark.parametrize("dims", [[2, 64, 64, 3], [3, 200, 200, 200, 1]], ids=lambda d: "x".join(map(str, d)))
def test_last_pass_of_half_the_waves(dims):
    """A last pass that at most half of the waves have a tile in is dealt over all workgroups: both sides of that line."""
    import torch
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    W, b = synth.siren_init(dims, 30.0, 3)
    m = dhq.Model(dims, 30.0, W, b)
    for n in (384 * cu, 384 * cu + 1):
        print(f"[calibrate] {dims} n={n}", flush=True)
        x = torch.rand((n, dims[0]), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda") * 2 - 1
        got, exp = _scales(m, x)
        assert np.array_equal(got, exp)
    m.close()


@pytest.mark.parametrize("n", [131072, 131073, 262145, 400001, 1048577], ids=["one_buffer", "two", "three_groups", "four_groups", "too_many_groups"])
def test_rows_beyond_the_buffers_room(n):
    """33 features take 64 bytes of codes; a buffer has 33 floats for each of 65 536 rows, two passes' worth of them."""
    import torch
    dims = [2, 33, 33, 33, 3]
    W, b = synth.siren_init(dims, 30.0, 6)
    m = dhq.Model(dims, 30.0, W, b)
    x = torch.rand((n, 2), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda") * 2 - 1
    print(f"[calibrate] {dims} n={n}", flush=True)
    got, exp = _scales(m, x)
    assert np.array_equal(got, exp)
    m.close()


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), 3.0e38, 1.0e32, float("nan")])
@pytest.mark.parametrize("dims,s0", [([2, 64, 64, 64, 3], None), ([2, 64, 64, 64, 3], 10.0), ([3, 256, 256, 256, 2], None), ([2, 200, 200, 1], 10.0)],
                         ids=["64", "64_wavelet", "256", "200_wavelet"])
def test_a_coordinate_beyond_the_range(dims, s0, value):
    """A scale without a bound makes activations that are no numbers: their codes, and the scales behind them, are the general path's."""
    import torch
    W, b = synth.siren_init(dims, 30.0, 5)
    m = dhq.Model(dims, 30.0, W, b, wavelet_s0=s0)
    x = torch.rand((5003, dims[0]), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda") * 2 - 1
    x[2501, 0] = value
    print(f"[calibrate] {dims} {s0} coordinate {value}", flush=True)
    got, exp = _scales(m, x)
    assert np.array_equal(got, exp, equal_nan=True)
    m.close()


@pytest.mark.parametrize("dims,s0,imag", [([2, 32, 32, 3], 1.0, 4.0), ([2, 32, 32, 32, 3], 0.5, 16.0), ([2, 128, 128, 3], 1.0, 8.0), ([2, 90, 90, 2], 0.8, 8.0),
                                          ([1, 16, 16, 1], 1.0, 8.0), ([2, 64, 64, 64, 3], 1.2, 4.0), ([3, 100, 3], 1.0, 8.0)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_complex_moduli_beyond_fp32(dims, s0, imag):
    """A wide envelope's modulus, up to exp(omega0^2 / 4 s0^2) = 2^325 at s0 = 1, is infinite at arguments of ordinary size.  The whole
    transform of such a coordinate is no number, which a maximum leaves out: with the other rows' the layer's scale is an ordinary
    one, and that coordinate's codes are the general path's."""
    import torch
    rng = np.random.default_rng(dims[1])
    W, b = synth.wire_init(dims, 30.0, 3)
    W[0] = (rng.uniform(-0.5, 0.5, W[0].shape) + 2j * imag * rng.uniform(-0.5, 0.5, W[0].shape)).astype(np.complex64)
    b[0] = b[0] * 0
    m = dhq.Model.complex_wavelet(dims, 30.0, W, b, s0, 8, 8)
    x = torch.rand((5003, dims[0]), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda") * 2 - 1
    corners = torch.sign(x[::50])
    x *= 1e-2 / imag
    x[::50] = corners
    print(f"[calibrate] complex {dims} s0={s0}", flush=True)
    got, exp = _scales(m, x)
    print(f"  scales {got}", flush=True)
    assert np.array_equal(got, exp, equal_nan=True)
    m.close()


@pytest.mark.parametrize("bias", [3.0e38, -3.0e38, 1.0e32])
@pytest.mark.parametrize("dims", [[2, 64, 64, 64, 3], [3, 200, 200, 2]], ids=lambda d: "x".join(map(str, d)))
def test_a_bias_beyond_the_range(dims, bias):
    """A feature whose argument is infinite or huge in every row: the codes of the layer's output are the general path's."""
    import torch
    W, b = synth.siren_init(dims, 30.0, 5)
    b[0][3] = bias
    m = dhq.Model(dims, 30.0, W, b)
    x = torch.rand((3001, dims[0]), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda") * 2 - 1
    print(f"[calibrate] {dims} bias {bias}", flush=True)
    got, exp = _scales(m, x)
    assert np.array_equal(got, exp, equal_nan=True)
    m.close()
