"""The refiner's input product in one launch for few tiles (gemm_fnr_kernel: 32- or 64-row tiles, two groups of wavefronts share
the ranges of K): single steps take it, passes of several steps add the same ranges inside the general product, and the
sums are added in the same order, so the containers are equal byte for byte."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


# D_h = 32 T
@pytest.mark.parametrize("B,T,H,d_e", [
    (33, 8, 128, 64),      # 2 ranges of two units of 64; a tile of one row, one column tile
    (65, 16, 256, 192),    # 4 ranges of two units
    (40, 40, 320, 64),     # 4 ranges of five units
    (130, 32, 256, 128),   # 8 ranges of two units
    (513, 16, 256, 1024),  # 64-row tiles, one row in the last; 4 ranges
    (1024, 32, 256, 1024), # 256 tiles of 64 rows: the most that take the launch; 2 ranges of eight units
])
def test_refiner_product_of_few_tiles(B, T, H, d_e, monkeypatch):
    need_gpu()
    import paper_2604_07239_amd as fa
    D, n = 32, B * (T + 24)
    blob = fi.init_blob(B, T, D, H, 5, std=0.05, d_e=d_e)
    src = fi.text(31, n)
    outs = []
    for steps in ("1", "8"):
        monkeypatch.setenv("FADE_STEPS_PER_PASS", steps)
        g = fa.Fade(fa.make_config(B, T, D, H, d_e=d_e, dtype=fa.BF16))
        g.load_weights(blob.data)
        outs.append(g.encode(src))
        np.testing.assert_array_equal(g.decode(outs[-1], n), src)
        g.close()
    assert outs[0].tobytes() == outs[1].tobytes()
