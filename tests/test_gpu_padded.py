"""Hidden widths that are no width of a whole-network kernel but round up to one: DHQ_AUTO runs them zero-padded."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from oracle import dhq_oracle as o
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu
OUT_TOL = 2e-3          # a coordinate without a code difference is within 1e-6 of the oracle; one with may move this far


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


# smallest and largest of each padded range, unequal widths with the same rounded-up one, every fan-in
SHAPES = [[3, 20, 20, 3], [1, 17, 1], [2, 33, 63, 48, 32], [4, 65, 128, 100, 5], [2, 200, 200, 200, 1], [3, 129, 255, 3],
          [2, 257, 257, 3], [1, 511, 300, 2], [4, 512, 363, 512, 32]]


@pytest.mark.parametrize("dims", SHAPES, ids=["x".join(map(str, d)) for d in SHAPES])
@pytest.mark.parametrize("s0", [None, 2.0], ids=["sine", "wavelet"])
def test_padded_widths(dims, s0):
    W, b = synth.siren_init(dims, 30.0, 5 + dims[1])
    rng = np.random.default_rng(dims[1])
    m = dhq.Model(dims, 30.0, W, b, wavelet_s0=s0)
    assert not m.has_fused()                               # DHQ_FUSED keeps to the exact widths
    for n in (1, 127, 257, 9000 + 7):
        print(f"[padded] {dims} s0={s0} n={n}", flush=True)
        x = rng.uniform(-1, 1, size=(n, dims[0])).astype(np.float32)
        net = o.quantize_net(dims, 30.0, 8, 8, W, b, gabor_s0=s0) if s0 is not None else o.quantize_net(dims, 30.0, 8, 8, W, b)
        exp = o.forward(net, x, calibrate=True)
        m.set_act_scales(net.s_a)
        auto, lw = _host(m.forward(_dev(x))), _host(m.forward(_dev(x), flags=dhq.DHQ_LAYERWISE))
        with pytest.raises(dhq.DhqError) as e:
            m.forward(_dev(x), flags=dhq.DHQ_FUSED)
        assert e.value.status == dhq.DHQ_EUNSUPPORTED
        err, err_lw = (np.abs(v.astype(np.float64) - exp).max(axis=1) for v in (auto, lw))
        print(f"  beyond {OUT_TOL}: {(err > OUT_TOL).sum()} (layer by layer {(err_lw > OUT_TOL).sum()}), max {err.max():.2e}, "
              f"median {np.median(err):.1e} ({np.median(err_lw):.1e}), rms {np.sqrt((err**2).mean()):.2e} "
              f"({np.sqrt((err_lw**2).mean()):.2e})", flush=True)
        assert (err > OUT_TOL).mean() <= max(3e-3, 1.0 / n) and err.max() <= 2e-2 and np.median(err) <= 1e-5
        # on-line scales: as the oracle's; up to 256 features one kernel per layer of the same arithmetic, so a static
        # forward with the measured scales gives the same bits
        dyn = _host(m.forward(_dev(x), flags=dhq.DHQ_DYNAMIC))
        s_dyn = m.dynamic_scales()
        rel = np.abs(s_dyn / net.s_a - 1)
        # Layers 0 and 1 see inputs without a quantizer's decision upstream that could differ on the maximum's coordinate
        # (or only layer 0's few codes); after that the coordinate that holds a layer's maximum may carry a code that fp32
        # and fp64 round differently.  One such code moves an input of the next layers by one step, 1 / 127 of the largest:
        # at most 1e-2 of the maximum.
        assert rel[:2].max() <= 1e-5 and rel.max() <= 1e-2
        if max(dims[1:-1]) <= 256:
            m.set_act_scales(s_dyn)
            assert np.array_equal(dyn, _host(m.forward(_dev(x))))
            out = _dev(np.zeros((n, dims[-1]), np.float32))
            if n <= dhq.dhq_noalloc_max_rows(m.handle):
                dhq.dhq_forward_noalloc(m.handle, _dev(x), out)
                assert np.array_equal(dyn, _host(out))
    m.close()


@pytest.mark.parametrize("width", [20, 200, 300])
def test_small_activations_keep_fp32_accuracy(width):
    """A wavelet layer whose envelope leaves only activations of 1e-6 .. 1e-3: what the transform loses in them has to stay relative to
    them, as it does in the layer-by-layer path's fp32 butterflies."""
    s0, dims = 10.0, [2, width, 3]
    rng = np.random.default_rng(width)
    W = [rng.uniform(-0.02, 0.02, (width, 2)).astype(np.float32), rng.uniform(-0.3, 0.3, (3, width)).astype(np.float32)]
    b = [rng.uniform(0.28, 0.32, width).astype(np.float32), np.zeros(3, np.float32)]
    x = rng.uniform(-1, 1, size=(20000, 2)).astype(np.float32)
    net = o.quantize_net(dims, 30.0, 8, 8, W, b, gabor_s0=s0)
    exp, dump = o.forward(net, x, calibrate=True, dump=True)
    assert 1e-5 < np.abs(dump.act[0]).max() < 2e-3
    m = dhq.Model(dims, 30.0, W, b, wavelet_s0=s0)
    m.set_act_scales(net.s_a)
    # a row is off where one of its Kp codes has fallen the other way, by half a code of the smaller weights at least; x^ in
    # codes (up to 127) is off by some 2^-23 * 127 = 1.5e-5 (the wavelet's own rounding and the sums'), so a row has such a
    # code with a probability of about 2 * 1.5e-5 * Kp, at most 1.6e-2; pieces with an absolute error of 2^-25 give a third and more
    code = float(net.s_a[1]) * float(net.s_w[1])
    off = {}
    for name, flags in (("auto", dhq.DHQ_AUTO), ("layer by layer", dhq.DHQ_LAYERWISE)):
        err = np.abs(_host(m.forward(_dev(x), flags=flags)).astype(np.float64) - exp).max(axis=1)
        off[name] = (err > 0.5 * code).mean()
    print(f"[padded] small activations, width {width}: rows with another code {off}", flush=True)
    assert max(off.values()) <= 2e-2
    m.close()


@pytest.mark.parametrize("dims_c", [[2, 181, 181, 3], [1, 20, 20, 1], [3, 45, 45, 45, 5], [4, 100, 100, 2]],
                         ids=["181", "20", "45", "100"])
def test_padded_complex_widths(dims_c):
    """Complex widths that are no power of two, on few rows and on many, against the oracle (the bounds of the complex networks: a
    differing code moves the output by about the network's own quantization error)."""
    Wc, bc = synth.wire_init(dims_c, 30.0, 11 + dims_c[1])
    dims, W, b = o.complex_net_to_real(dims_c, Wc, bc)
    m = dhq.Model.complex_wavelet(dims_c, 30.0, Wc, bc, 10.0)
    rng = np.random.default_rng(dims_c[1])
    for n in (1, 33, 300, 9007):
        print(f"[padded] complex {dims_c} n={n}", flush=True)
        x = rng.uniform(-1, 1, size=(n, dims_c[0])).astype(np.float32)
        net = o.quantize_net(dims, 30.0, 8, 8, W, b, gabor_s0=o.ComplexSpread(10.0))
        exp = o.forward(net, x, calibrate=True)
        ref, _ = o.mlp_float(dims, 30.0, W, b, x, want_f32=False, gabor_s0=o.ComplexSpread(10.0))
        m.set_act_scales(net.s_a)
        auto, lw = _host(m.forward(_dev(x))), _host(m.forward(_dev(x), flags=dhq.DHQ_LAYERWISE))
        for v in (auto, lw):
            err = np.abs(v.astype(np.float64) - exp).max(axis=1)
            print(f"  beyond {OUT_TOL}: {(err > OUT_TOL).sum()}, max {err.max():.2e}, median {np.median(err):.1e}", flush=True)
            assert (err > OUT_TOL).mean() <= max(3e-3, 1.0 / n)
            assert err.max() <= max(2e-2, 10 * np.sqrt(np.mean((exp - ref) ** 2))) and np.median(err) <= 1e-5
    m.close()


def test_padded_cosine_keeps_the_layer_by_layer_path():
    """A wavelet without an envelope (s0 = 0) is 1 at 0: no padded feature can come out as zero."""
    dims = [2, 40, 40, 3]
    W, b = synth.siren_init(dims, 30.0, 3)
    m = dhq.Model(dims, 30.0, W, b, wavelet_s0=0.0)
    x = _dev(np.random.default_rng(0).uniform(-1, 1, size=(999, 2)).astype(np.float32))
    m.calibrate(x)
    assert np.array_equal(_host(m.forward(x)), _host(m.forward(x, flags=dhq.DHQ_LAYERWISE)))
    m.close()


@pytest.mark.parametrize("dims,mode,n", [([2, 200, 200, 1], dhq.DHQ_ROTATE_IN, 5000), ([3, 200, 200, 1], dhq.DHQ_ROTATE_IN, 70001),
                                         ([2, 64, 64, 3], dhq.DHQ_ROTATE_BOTH, 140001), ([2, 33, 33, 3], dhq.DHQ_ROTATE_IN, 150000)],
                         ids=["one_chunk", "chunks", "two_sided", "beyond_the_codes_room"])
def test_calibrated_scales_are_the_dynamic_ones(dims, mode, n):
    """Calibration on one chunk, on several with the codes kept between the layers, and on more rows than the codes have
    room for (33 features: 64 code bytes against 132 of floats, 135 168 rows): the on-line scales of the layer-by-layer
    path, bit for bit."""
    W, b = synth.siren_init(dims, 30.0, 17)
    m = dhq.Model(dims, 30.0, W, b, mode=mode)
    x = _dev(np.random.default_rng(n).uniform(-1, 1, size=(n, dims[0])).astype(np.float32))
    m.calibrate(x)
    s_cal = m.scales()[1]
    m.forward(x, flags=dhq.DHQ_LAYERWISE | dhq.DHQ_DYNAMIC)
    assert np.array_equal(s_cal, m.dynamic_scales())
    m.close()
