"""The whole-network kernels on few rows, and on what is left of a last pass: every way the rows can be dealt to workgroups and
waves gives a coordinate the same bits."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["sine", "wavelet", "complex"])
@pytest.mark.parametrize("width", [32, 64, 128, 256, 200, 90])
def test_same_bits_however_the_rows_are_dealt(width, act):
    import torch
    torch.cuda.set_device(0)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    if act == "complex":
        dims = [2, width // 2, width // 2, 3]
        W, b = synth.wire_init(dims, 30.0, width)
        m = dhq.Model.complex_wavelet(dims, 30.0, W, b, 10.0)
    else:
        dims = [3, width, width, width, 5]
        W, b = synth.siren_init(dims, 30.0, width)
        m = dhq.Model(dims, 30.0, W, b, wavelet_s0=10.0 if act == "wavelet" else None)
    g = torch.Generator(device="cuda").manual_seed(width)
    n_all = 32 * cu * 12                                    # one full pass and a half
    x = torch.rand((n_all, dims[0]), generator=g, device="cuda") * 2 - 1
    m.calibrate(x)
    ref = m.forward(x).cpu().numpy()
    assert np.isfinite(ref).all() and np.abs(ref).max() > 1e-3
    # in 32-row tiles per CU: the ends of every range the launch tells apart, alone and after a full pass, and ragged rows
    for tiles in (1, 2 * cu, 2 * cu + 1, 3 * cu, 3 * cu + 1, 4 * cu, 4 * cu + 1, 8 * cu, 8 * cu + 1, 9 * cu, 9 * cu + 1, 10 * cu, 10 * cu + 1, 11 * cu):
        for ragged in (0, 31):
            n = 32 * tiles - ragged
            print(f"[few rows] {act} {width} n={n}", flush=True)
            out = m.forward(x[:n]).cpu().numpy()
            assert np.array_equal(out, ref[:n])
    # after more full passes than dealing a last one pays for: a few and most of its waves busy, and whole passes
    for n in (32 * cu * 8 * 12 + 77, 32 * cu * 8 * 11 + 32 * cu * 6 - 5, 32 * cu * 8 * 12):
        print(f"[few rows] {act} {width} n={n}", flush=True)
        out = m.forward(x.repeat((n + n_all - 1) // n_all, 1)[:n].contiguous()).cpu().numpy()
        for i in range(0, n, n_all):
            assert np.array_equal(out[i:i + n_all], ref[:min(n_all, n - i)])
    m.close()
