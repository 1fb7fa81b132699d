"""Fan-ins of 5 to 64 on the whole-network kernels under DHQ_AUTO: the input's codes come from the layer-by-layer path's transform."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
import test_gpu_padded as padded
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu


# rotated inputs of 8, 16, 32 and 64 codes (one and two k blocks), exact and padded widths of every kernel; beyond them layer by layer
@pytest.mark.parametrize("dims", [[5, 32, 32, 3], [9, 20, 20, 1], [12, 64, 64, 3], [33, 50, 50, 3], [40, 128, 128, 2], [16, 90, 90, 90, 5],
                                  [64, 256, 256, 3], [17, 200, 140, 3], [5, 512, 512, 3], [32, 300, 300, 2], [40, 32, 32, 3], [40, 512, 512, 3],
                                  [65, 64, 64, 3]], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("s0", [None, 2.0], ids=["sine", "wavelet"])
def test_against_oracle(dims, s0):
    """The gates of the padded networks (DHQ_FUSED refused, on-line scales layer by layer)."""
    import torch
    from oracle import dhq_oracle as o
    W, b = synth.siren_init(dims, 30.0, 5 + dims[1])
    rng = np.random.default_rng(dims[0])
    m = dhq.Model(dims, 30.0, W, b, wavelet_s0=s0)
    assert not m.has_fused()
    for n in (1, 31, 257, 9007):
        print(f"[wide input] {dims} s0={s0} n={n}", flush=True)
        x = rng.uniform(-1, 1, size=(n, dims[0])).astype(np.float32)
        net = o.quantize_net(dims, 30.0, 8, 8, W, b, gabor_s0=s0) if s0 is not None else o.quantize_net(dims, 30.0, 8, 8, W, b)
        exp = o.forward(net, x, calibrate=True)
        m.set_act_scales(net.s_a)
        auto, lw = (padded._host(m.forward(padded._dev(x), flags=f)) for f in (dhq.DHQ_AUTO, dhq.DHQ_LAYERWISE))
        with pytest.raises(dhq.DhqError) as e:
            m.forward(padded._dev(x), flags=dhq.DHQ_FUSED)
        assert e.value.status == dhq.DHQ_EUNSUPPORTED
        err, err_lw = (np.abs(v.astype(np.float64) - exp).max(axis=1) for v in (auto, lw))
        print(f"  beyond {padded.OUT_TOL}: {(err > padded.OUT_TOL).sum()} (layer by layer {(err_lw > padded.OUT_TOL).sum()}), max {err.max():.2e}, "
              f"median {np.median(err):.1e} ({np.median(err_lw):.1e})", flush=True)
        assert (err > padded.OUT_TOL).mean() <= max(3e-3, 1.0 / n) and err.max() <= 2e-2 and np.median(err) <= 1e-5
        dyn = padded._host(m.forward(padded._dev(x), flags=dhq.DHQ_DYNAMIC))
        assert np.array_equal(dyn, padded._host(m.forward(padded._dev(x), flags=dhq.DHQ_DYNAMIC | dhq.DHQ_LAYERWISE)))
        m.calibrate(padded._dev(x))
        assert np.array_equal(m.scales()[1], m.dynamic_scales())
    m.close()


@pytest.mark.parametrize("dims", [[5, 32, 32, 3], [9, 20, 20, 1], [33, 50, 50, 3], [12, 64, 64, 64, 3], [40, 128, 100, 2], [16, 90, 90, 90, 5], [64, 256, 256, 3],
                                  [17, 200, 140, 3], [5, 180, 180, 180, 2], [5, 512, 512, 512, 3], [32, 300, 400, 2], [9, 257, 257, 32]],
                         ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("act", ["sine", "wavelet", "complex"])
@pytest.mark.parametrize("bits", [8, 4])
def test_same_bits_as_layer_by_layer(dims, act, bits):
    """Whichever kernels run: rows at the edges of a wave's and a workgroup's tile, coordinates far outside and not finite."""
    import torch
    if act == "complex":
        dims = [dims[0]] + [max(1, d // 2) for d in dims[1:-1]] + [dims[-1]]
        W, b = synth.wire_init(dims, 30.0, 3)
        m = dhq.Model.complex_wavelet(dims, 30.0, W, b, 10.0, bits, bits)
    else:
        W, b = synth.siren_init(dims, 30.0, 3)
        m = dhq.Model(dims, 30.0, W, b, bits, bits, wavelet_s0=10.0 if act == "wavelet" else None)
    x = torch.rand((70001, dims[0]), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda") * 2 - 1
    m.calibrate(x[:3000].contiguous())
    x[5, 0], x[77, -1], x[300, 1], x[301, 2], x[4000] = float("inf"), float("nan"), -float("inf"), 3e38, 0.0
    for n in (1, 31, 33, 257, 9007, 70001):
        print(f"[wide input] {dims} {act} {bits} bits n={n}", flush=True)
        auto, lw = (m.forward(x[:n].contiguous(), flags=f) for f in (dhq.DHQ_AUTO, dhq.DHQ_LAYERWISE))
        assert torch.equal(auto.view(torch.int32), lw.view(torch.int32))
    m.close()


def test_rows_beyond_the_workspace_and_every_tile():
    """A coordinate's value does not depend on where it sits: in several workspaces full of codes, in full passes and their rest."""
    import torch
    for dims in ([12, 64, 64, 3], [40, 200, 200, 1], [20, 300, 300, 3]):
        W, b = synth.siren_init(dims, 30.0, 8)
        m = dhq.Model(dims, 30.0, W, b)
        room = 65536 * max(64, 1 << (dims[1] - 1).bit_length()) // (1 << (dims[0] - 1).bit_length())
        n = 2 * room + 1000
        print(f"[wide input] {dims} n={n}", flush=True)
        x = torch.rand((n, dims[0]), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda") * 2 - 1
        m.calibrate(x[:4000].contiguous())
        out = m.forward(x)
        for lo, hi in ((0, 40), (room - 50, room + 50), (2 * room - 7, 2 * room + 300), (n - 33, n)):
            assert torch.equal(out[lo:hi], m.forward(x[lo:hi].contiguous()))
        m.close()
