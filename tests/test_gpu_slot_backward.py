"""The newest-slot backward where a batch of W_m's rows ends inside the slot (12 columns) and a workgroup's streams past the last one,
with one and with two streams per wavefront: gradients of the first update against the oracle, bar of the other bf16 gradients."""
import numpy as np
import pytest

from gpu_helpers import need_gpu
from test_gpu_online import _compare_gradients, _make_pair_with_wu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 37, 2051])
def test_slot_gradients_at_edges(B):
    torch = need_gpu()
    T, D, H = 16, 32, 192
    g, o, blob = _make_pair_with_wu_grad(B, T, D, H, "bf16", seed=17, update_mode=1, randomize=True, std=0.05)
    data = np.random.default_rng(B).integers(0, 256, (B, T + 1), dtype=np.uint8)
    win, tgt = np.ascontiguousarray(data[:, :T]), np.ascontiguousarray(data[:, T])
    g.step_probs(torch.from_numpy(win).cuda(), None, None, None)
    o.step_probs(win, None)
    go = o.backward(tgt, None)
    g.step_update(torch.from_numpy(tgt).cuda(), None)
    _compare_gradients(blob, g.debug_grad(), go, 3e-2, f"B={B}")
