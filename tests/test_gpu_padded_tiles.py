"""Padded networks leave out tiles that are all padding: every number of tiles, on both sides of each step."""
import pytest

import test_gpu_padded as padded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [[2, 96, 96, 3], [1, 97, 97, 97, 2], [2, 160, 129, 160, 3], [3, 161, 192, 1], [2, 193, 224, 193, 3], [4, 225, 225, 3],
                                  [2, 320, 320, 320, 3], [3, 321, 257, 384, 1], [2, 384, 384, 3], [1, 385, 300, 385, 2], [2, 448, 448, 448, 3],
                                  [4, 449, 449, 32]], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("s0", [None, 2.0], ids=["sine", "wavelet"])
def test_every_number_of_tiles(dims, s0):
    padded.test_padded_widths(dims, s0)
