"""Where a reset takes the loaded weights from: the copy on the device, or host memory on a card too full for it. Same results."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B", [("bf16", 37), ("f32", 5), ("f32", 260)])
def test_reset_from_device_or_host_copy(dtype, B, monkeypatch):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    T, D, H = 8, 32, 64
    blobs = [fi.init_blob(B, T, D, H, seed, std=0.05).data for seed in (5, 6)]
    data = torch.from_numpy(np.random.default_rng(B).integers(0, 256, (B, T + 1), dtype=np.uint8)).cuda()
    src = fi.text(4, B * (T + 6) - 3)
    got = []
    for host in ("0", "1"):
        monkeypatch.setenv("FADE_RESTORE_FROM_HOST", host)
        g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16 if dtype == "bf16" else fa.F32, update_mode=fa.ONLINE_ADAM))
        out = []
        for blob in blobs:  # the first load gives the device copy up at its end, the second one finds none
            g.load_weights(blob)
            for _ in range(2):
                g.step_probs(data[:, :T].contiguous())
                g.step_update(data[:, T].contiguous())
            out.append(g.get_weights())
            assert (out[-1] != blob).any()
            g.reset()
            np.testing.assert_array_equal(g.get_weights(), blob)
            out.append(g.encode(src))
            np.testing.assert_array_equal(g.decode(out[-1], src.size), src)
        got.append(out)
        g.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


def test_a_request_that_does_not_fit_leaves_a_working_context():
    """A job whose payload buffer exceeds any card: the device copy of the weights is given up for it, the call fails with
    FADE_E_OOM before it launches anything on the job, and the context codes the next one as before, from the host copy."""
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 512, 8, 32, 64  # 9 MB of weights
    blob = fi.init_blob(B, T, D, H, 5, std=0.05).data
    src = fi.text(4, B * (T + 6) - 3)
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, update_mode=fa.ONLINE_ADAM))
    g.load_weights(blob)
    want = g.encode(src)
    job = torch.zeros(16, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for _ in range(2):  # the second time there is no device copy left to give up
        with pytest.raises(fa.FadeError) as e:
            g.encode_device(job, 1 << 40)
        assert e.value.code == -8
    assert torch.cuda.mem_get_info()[0] >= before + (4 << 20)
    np.testing.assert_array_equal(g.encode(src), want)
    np.testing.assert_array_equal(g.decode(want, src.size), src)
    g.reset()
    np.testing.assert_array_equal(g.get_weights(), blob)
    g.close()
