"""The weights on their way to the host: pinned chunks, several host threads (fade_get_weights of adapting contexts)."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,T,D,H,level", [("f32", 1, 16, 16, 64, 0),     # less than one chunk
                                                  ("f32", 5, 32, 16, 128, 0),    # the scalars leave no run aligned alike in blob and layout
                                                  ("bf16", 67, 64, 32, 128, 0),  # ten chunks and more than threads, the last one ragged
                                                  ("bf16", 3, 16, 32, 128, 2)])
def test_weights_come_back_as_loaded(dtype, B, T, D, H, level):
    need_gpu()
    import paper_2604_07239_amd as fa
    blob = fi.init_blob(B, T, D, H, seed=B)
    data = np.random.default_rng(B).standard_normal(blob.data.size).astype(np.float32)  # every element its own value
    ctx = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16 if dtype == "bf16" else fa.F32, update_mode=fa.ONLINE_ADAM, ablation=level))
    ctx.load_weights(data)
    for _ in range(3):  # the buffers are used again and again
        assert np.array_equal(ctx.get_weights(), data)
