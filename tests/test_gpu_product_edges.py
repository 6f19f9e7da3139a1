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


@pytest.mark.parametrize("B,d_e", [(37, 2112), (130, 4160)])  # 66 and 130 blocks of 64 along K = 2 D_e: two ranges, where four or eight do not divide
def test_wide_refiner_whose_contraction_divides_into_few_ranges(B, d_e):
    torch = need_gpu()
    from test_gpu_online import _compare_gradients, _make_pair_with_wu_grad
    T, D, H = 8, 32, 64
    g, o, blob = _make_pair_with_wu_grad(B, T, D, H, "bf16", seed=B, update_mode=1, std=0.05, d_e=d_e)
    data = np.random.default_rng(B).integers(0, 256, (B, T + 1), dtype=np.uint8)
    win, tgt = np.ascontiguousarray(data[:, :T]), np.ascontiguousarray(data[:, T])
    g.step_probs(torch.from_numpy(win).cuda())
    o.step_probs(win, None)
    go = o.backward(tgt, None)
    g.step_update(torch.from_numpy(tgt).cuda())
    _compare_gradients(blob, g.debug_grad(), go, 3e-2, f"D_e={d_e}")
    g.close()
