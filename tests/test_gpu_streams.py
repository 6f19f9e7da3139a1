"""What the calls wait for, and which streams they touch."""
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
