"""What the calls wait for, which streams they touch, and how a caller's buffer may lie."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
def test_reset_returns_when_the_stream_is_idle(mode):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 5, 8, 32, 64
    s = torch.cuda.Stream()
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, update_mode=mode, hip_stream=s.cuda_stream))
    g.load_weights(fi.init_blob(B, T, D, H, 3).data)
    with torch.cuda.stream(s):
        torch.cuda._sleep(200_000_000)  # some 100 ms in front of the reset
    assert not s.query()
    g.reset()
    assert s.query()
    g.close()


def test_load_weights_does_not_wait_for_other_streams():
    """A program that works on the default stream may load a model on another one meanwhile."""
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 5, 8, 32, 64
    s = torch.cuda.Stream()
    blob = fi.init_blob(B, T, D, H, 3)
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, hip_stream=s.cuda_stream))
    g.load_weights(np.zeros_like(blob.data))  # everything that a first call sets up is there
    torch.cuda.synchronize()
    torch.cuda._sleep(400_000_000)
    g.load_weights(blob.data)
    assert not torch.cuda.default_stream().query()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(g.get_weights(), blob.data)
    g.close()


@pytest.mark.parametrize("dtype,mode", [("bf16", 0), ("bf16", 1), ("f32", 0), ("f32", 1)])
@pytest.mark.parametrize("at", [1, 2, 3])
def test_probabilities_to_a_buffer_between_two_16_byte_pieces(dtype, mode, at):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 5, 8, 32, 64
    blob = fi.init_blob(B, T, D, H, 3, std=0.05)
    win = torch.from_numpy(np.random.default_rng(1).integers(0, 256, (B, T), dtype=np.uint8)).cuda()
    got = []
    for shift in (0, at):
        g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16 if dtype == "bf16" else fa.F32, update_mode=mode))
        g.load_weights(blob.data)
        buf = torch.full((B * 256 + 8,), -1.0, device="cuda")
        g.step_probs(win, None, None, buf[shift:shift + B * 256])
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        assert (host[:shift] == -1).all() and (host[shift + B * 256:] == -1).all()
        got.append(host[shift:shift + B * 256])
        g.close()
    np.testing.assert_array_equal(got[0], got[1])
