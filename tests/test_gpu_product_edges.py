"""The 256 x 256 product at its shortest and odd contractions: a pass of 64 steps of 256 streams (16384 rows) takes it, single
steps take the small tiles, and both add the same k-steps in the same order, so the containers are equal byte for byte."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


# contractions of 4, 5, 7 and 13 units of 64: every phase of the three-slot ring of units at its end
@pytest.mark.parametrize("d_cache,d_e", [(256, 448), (320, 256), (832, 320)])
def test_large_tile_contraction_lengths(d_cache, d_e, monkeypatch):
    need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, n = 256, 32, 32, 256 * (32 + 128)
    blob = fi.init_blob(B, T, D, d_cache, 5, std=0.05, d_cache=d_cache, d_e=d_e)
    src = fi.text(27, n)
    outs = []
    for steps in ("1", "64"):
        monkeypatch.setenv("FADE_STEPS_PER_PASS", steps)
        g = fa.Fade(fa.make_config(B, T, D, d_cache, d_cache=d_cache, d_e=d_e, dtype=fa.BF16))
        g.load_weights(blob.data)
        outs.append(g.encode(src))
        np.testing.assert_array_equal(g.decode(outs[-1], n), src)
        g.close()
    assert outs[0].tobytes() == outs[1].tobytes()
