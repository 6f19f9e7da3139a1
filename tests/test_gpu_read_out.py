"""The weights on their way to the host: pinned chunks, several host threads (fade_get_weights of adapting contexts)."""
import numpy as np
import pytest

import fade_inputs as fi
from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,T,D,H,level", [("f32", 1, 16, 16, 64, 0),     # two chunks, the second one short
                                                  ("f32", 5, 32, 16, 128, 0),    # the scalars leave no run aligned alike in blob and layout
                                                  ("bf16", 67, 64, 32, 128, 0),  # 41 chunks, the last one ragged
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


def test_weights_behind_work_on_the_callers_per_thread_stream():
    """hipStreamPerThread as the context's stream: every thread has its own, and the read-out waits for the caller's."""
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 128, 16, 32, 128  # six chunks
    blob = fi.init_blob(B, T, D, H, 3)
    text = np.random.default_rng(5).integers(0, 256, (B, T + 1), dtype=np.uint8)
    win, tgt = torch.from_numpy(np.ascontiguousarray(text[:, :T])).cuda(), torch.from_numpy(np.ascontiguousarray(text[:, T])).cuda()
    torch.cuda.synchronize()
    got = []
    for handle in (0, 2):  # a stream of the library's own; hipStreamPerThread
        g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, update_mode=fa.ONLINE_ADAM, hip_stream=handle))
        g.load_weights(blob.data)
        if handle:
            with torch.cuda.stream(torch.cuda.ExternalStream(handle)):
                torch.cuda._sleep(200_000_000)  # some 100 ms in front of the step
        g.step_probs(win)
        g.step_update(tgt)
        got.append(g.get_weights())
        g.close()
    assert not np.array_equal(got[0], blob.data)
    assert np.array_equal(got[0], got[1])


def test_weights_do_not_join_a_graph():
    """A read-out while the context's stream is captured is refused and leaves nothing in the graph."""
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, D, H = 1, 16, 16, 64
    blob = fi.init_blob(B, T, D, H, 3)
    s = torch.cuda.Stream()
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.F32, update_mode=fa.ONLINE_ADAM, hip_stream=s.cuda_stream))
    g.load_weights(blob.data)
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        graph.capture_begin()
        x.add_(1.0)
        with pytest.raises(fa.FadeError):
            g.get_weights()
        graph.capture_end()
        for k in (1, 2):
            graph.replay()
            s.synchronize()
            assert float(x.sum()) == 64.0 * k
    assert np.array_equal(g.get_weights(), blob.data)
    g.close()
