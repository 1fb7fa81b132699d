"""Two-sided networks on few rows: one M tile per wave, with the bits of the kernel for many rows."""
import numpy as np
import pytest

import paper_2508_13478_amd as dhq
from paper_2508_13478_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [32, 64, 128, 256])
@pytest.mark.parametrize("s0,bits", [(None, 8), (10.0, 8), (None, 4)], ids=["sine", "wavelet", "4_bits"])
def test_few_rows_have_the_bits_of_many(width, s0, bits):
    """Rows at the edges of a wave's tile, one to five 32-row tiles per CU of 256, and a full pass with such a rest."""
    import torch
    dims = [3, width, width, width, 5]
    W, b = synth.siren_init(dims, 30.0, width)
    m = dhq.Model(dims, 30.0, W, b, bits, bits, mode=dhq.DHQ_ROTATE_BOTH, wavelet_s0=s0)
    x = torch.rand((65536 + 8192 * 5, 3), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda") * 2 - 1
    m.calibrate(x[:5000].contiguous())
    big = m.forward(x[:65536].contiguous())  # a full pass
    for n in (1, 31, 33, 1000, 8192, 8193, 24576, 40960):
        print(f"[two-sided] width {width} s0={s0} n={n}", flush=True)
        assert torch.equal(m.forward(x[:n].contiguous()), big[:n])
        rest = m.forward(x[:65536 + n].contiguous())
        assert torch.equal(rest[:65536], big) and torch.equal(rest[65536:], m.forward(x[65536:65536 + n].contiguous()))
    m.close()
