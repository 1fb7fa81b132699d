"""On-line scales on the per-layer kernels: whether the launches pass floats or codes, at the ends of every range of rows that the
launch tells apart, a forward gives what a static forward with the scales it measured gives, bit for bit."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu

# 256ths of the CUs up to which the first, second and third pass go on floats: the rows on either side of each line
LINES = {("sine", 32): (104, 0, 0), ("sine", 64): (120, 0, 0), ("sine", 128): (62, 0, 0), ("sine", 256): (80, 0, 0),
         ("wavelet", 32): (176, 192, 32), ("wavelet", 64): (136, 0, 0), ("wavelet", 128): (110, 0, 0), ("wavelet", 256): (120, 112, 0),
         ("complex", 32): (176, 160, 200), ("complex", 64): (200, 48, 0), ("complex", 128): (168, 0, 0), ("complex", 256): (128, 0, 0)}


def _model(act, width, seed):
    if act == "complex":
        dims_c = [2, width // 2, 3]
        W, b = synth.wire_init(dims_c, 30.0, seed)
        return dhq.Model.complex_wavelet(dims_c, 30.0, W, b, 10.0)
    dims = [2, width, width, 3]
    W, b = synth.siren_init(dims, 30.0, seed)
    return dhq.Model(dims, 30.0, W, b, wavelet_s0=10.0 if act == "wavelet" else None)


@pytest.mark.parametrize("act", ["sine", "wavelet", "complex"])
@pytest.mark.parametrize("width", [32, 64, 128, 256, 26, 100, 200])
def test_floats_and_codes_give_the_same_bits(width, act):
    import torch
    torch.cuda.set_device(0)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    nf = 1 << (width - 1).bit_length()
    rows = {1, 129, 300, 256 * cu, 256 * cu + 1, 512 * cu + 1, 900}
    rows |= {384 * cu, 384 * cu + 1}  # a last pass that half of the waves have a tile in (dealt over all workgroups), and one tile more
    for p, line in enumerate(LINES[(act, nf)]):
        if line:
            n = 256 * (p * cu + line * cu // 256)
            rows |= {n - 31, n, n + 1}
    rows = sorted(rows)
    m = _model(act, width, width)
    g = torch.Generator(device="cuda").manual_seed(width)
    x = torch.rand((rows[-1], 2), generator=g, device="cuda") * 2 - 1
    dhq.dhq_reserve_dynamic(m.handle, rows[len(rows) // 2])  # the later ones grow the workspace
    for n in rows:
        print(f"[dynamic rows] {act} {width} n={n}", flush=True)
        dyn = m.forward(x[:n], flags=dhq.DHQ_DYNAMIC)
        s_a = m.dynamic_scales()
        m.set_act_scales(s_a)
        ref = m.forward(x[:n])
        assert torch.equal(dyn, ref) and bool(torch.isfinite(ref).all()) and float(ref.abs().max()) > 1e-3
        if n <= dhq.dhq_noalloc_max_rows(m.handle):
            out = torch.zeros_like(ref)
            dhq.dhq_forward_noalloc(m.handle, x[:n], out)
            assert torch.equal(out, ref) and np.array_equal(s_a, m.dynamic_scales())
    m.close()


def test_noalloc_at_its_row_limit():
    """The most rows the fixed scratch takes, for padded widths whose rows are wider than their activations."""
    import torch
    torch.cuda.set_device(0)
    for width in (129, 200, 65, 40, 17):
        m = _model("sine", width, 3)
        n = dhq.dhq_noalloc_max_rows(m.handle)
        print(f"[noalloc limit] {width} n={n}", flush=True)
        x = torch.rand((n, 2), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda") * 2 - 1
        out = torch.zeros((n, 3), device="cuda")
        dhq.dhq_forward_noalloc(m.handle, x, out)
        s_a = m.dynamic_scales()
        assert torch.equal(out, m.forward(x, flags=dhq.DHQ_DYNAMIC)) and np.array_equal(s_a, m.dynamic_scales())
        m.close()
