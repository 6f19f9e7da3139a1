"""Weights and optimiser state past the caches (nt loads and stores, bf16 path, chosen by size) or through them: a hint to the memory
system that may change no bit of probabilities or adapted weights. The fp32 path has no such access: there the override does nothing."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


# one stream; more streams than a workgroup of the per-stream product takes, not a multiple of them; a wide slot; frozen weights
@pytest.mark.parametrize("dtype,B,online,widths", [("bf16", 1, 1, {}), ("bf16", 37, 1, {}), ("bf16", 66, 1, dict(d_cache=512, d_e=128)),
                                                   ("bf16", 37, 0, {}), ("f32", 37, 1, {}), ("f32", 259, 1, {})])
def test_same_bits_streamed_or_cached(dtype, B, online, widths, monkeypatch):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    T, D, H, steps = 8, 32, 64, 4
    blob = fi.init_blob(B, T, D, H, 5, std=0.05, **widths)
    data = torch.from_numpy(np.random.default_rng(B).integers(0, 256, (B, T + steps), dtype=np.uint8)).cuda()
    got = []
    for streamed in ("0", "1"):
        monkeypatch.setenv("FADE_STREAMED", streamed)
        g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16 if dtype == "bf16" else fa.F32,
                                   update_mode=fa.ONLINE_ADAM if online else fa.FROZEN, **widths))
        g.load_weights(blob.data)
        probs = torch.zeros((steps, B, 256), device="cuda")
        for i in range(steps):
            g.step_probs(data[:, i:i + T].contiguous(), None, None, probs[i])
            if online:
                g.step_update(data[:, i + T].contiguous())
        torch.cuda.synchronize()
        got.append((probs.cpu().numpy(), g.get_weights()))
        g.close()
    assert np.isfinite(got[0][0]).all()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
