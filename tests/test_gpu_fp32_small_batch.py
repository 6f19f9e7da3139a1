"""The fp32 kernels of small batches (16 x 16 tiles, products sharing a launch, weight gradients with their Adam step) at the
sizes where a tile, a strip or a batch of loads ends: against the oracle at the fp32 bars of the other parity tests."""
import numpy as np
import pytest

from gpu_helpers import make_pair, need_gpu
from test_gpu_online import _grad_check
from test_gpu_parity import _step_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,H,widths", [
    (1, 8, 16, 64, {}),                                   # one row of a tile, D_h = 128
    (17, 8, 32, 64, {}),                                  # one row of a second tile, 32 channels
    (31, 64, 16, 64, dict(d_cache=320)),                  # slots of five: no 16-byte pieces
    (256, 8, 16, 64, {}),                                 # the most streams these kernels take
    (5, 128, 16, 128, dict(d_cache=2048, d_e=2048)),      # D_h = D_cache = D_e = 2048: several batches of loads, rows of 128 partial sums
])
def test_step_parity_at_tile_edges(B, T, D, H, widths):
    _step_parity(B, T, D, H, "f32", steps=3, randomize=True, seed=70 + B, **widths)


# 2e-4 as elsewhere. 4e-4 at D_h = 2048: the second update starts from two states that Adam's sign-like first step has moved apart
# by up to 2 lr wherever a gradient lies within fp32's error of zero (test_first_and_second_update_at_2048_channels shows both parts).
@pytest.mark.parametrize("B,T,D,H,tol,widths", [
    (1, 8, 16, 64, 2e-4, {}),
    (15, 8, 32, 64, 2e-4, {}),
    (17, 16, 16, 64, 2e-4, dict(d_cache=64, d_e=192)),    # 272 tokens: a third, short chunk of the conv gradient
    (6, 64, 16, 64, 2e-4, dict(d_cache=320)),             # slots of five: strips without 16-byte pieces
    (33, 8, 16, 128, 2e-4, dict(d_cache=256)),            # slots of 32: two column tiles of the newest-slot backward
    (4, 128, 16, 128, 4e-4, {}),                          # D_h = 2048
])
def test_gradients_and_adam_at_tile_edges(B, T, D, H, tol, widths):
    _grad_check("f32", B, T, D, H, seed=90 + B, tol=tol, **widths)


def test_update_without_active_streams():
    """A gradient of zero in every shared tensor (not the previous update's), and weights that stay as they are, to the bit."""
    torch = need_gpu()
    B, T, D, H = 7, 8, 16, 64
    g, _, blob = make_pair(B, T, D, H, "f32", seed=21, update_mode=1, std=0.05)
    data = torch.from_numpy(np.random.default_rng(3).integers(0, 256, (B, T + 1), dtype=np.uint8)).cuda()
    g.step_probs(data[:, :T].contiguous())
    g.step_update(data[:, T].contiguous())
    before = g.get_weights()
    assert np.abs(blob.view(g.debug_grad(), "W_r")).max() > 0
    none = torch.zeros(B, dtype=torch.uint8, device="cuda")
    g.step_probs(data[:, :T].contiguous(), none)
    g.step_update(data[:, T].contiguous(), none)
    grad = g.debug_grad()
    for name, _, _ in blob.specs:
        assert name == "W_U" or not blob.view(grad, name).any(), name
    np.testing.assert_array_equal(g.get_weights(), before)
    g.close()


@pytest.mark.parametrize("rows16", ["1", "0"])
@pytest.mark.parametrize("seed", [94, 95])
def test_first_and_second_update_at_2048_channels(seed, rows16, monkeypatch):
    """Four streams, D_h = 2048, with the small-batch kernels and with the general ones: what the kernels' arithmetic leaves of a
    gradient's error, and what the two states' drift adds to the second one."""
    torch = need_gpu()
    monkeypatch.setenv("FADE_DEBUG_WU_GRAD", "1")
    monkeypatch.setenv("FADE_F32_ROWS16", rows16)
    B, T, D, H = 4, 128, 16, 128
    g, o, blob = make_pair(B, T, D, H, "f32", seed=seed, update_mode=1, randomize=True, std=0.05)
    data = np.random.default_rng(seed).integers(0, 256, (B, T + 3), dtype=np.uint8)
    worst = []
    for i in range(2):
        win, tgt = np.ascontiguousarray(data[:, i:i + T]), np.ascontiguousarray(data[:, i + T])
        g.step_probs(torch.from_numpy(win).cuda())
        o.step_probs(win, None)
        want = o.backward(tgt, None)
        g.step_update(torch.from_numpy(tgt).cuda())
        got = g.debug_grad()
        o.step_update(tgt, None)
        worst.append(max((float(np.abs(blob.view(got, n).astype(np.float64) - blob.view(want, n)).max() / np.abs(blob.view(want, n)).max()), n)
                         for n, shape, _ in blob.specs if blob.view(got, n).size > 1))
    print(f"D_h = 2048, seed {seed}, small-batch kernels {rows16}: first update {worst[0]}, second {worst[1]}", flush=True)
    # From identical states: a chain of products of up to 2048 terms, sqrt(2048) 2^-24 = 2.7e-6 each, a few of them in a row (measured
    # 0.9-1.6e-6 with the small-batch kernels, 3-6e-6 with the general ones). From states that drifted: 2.8e-4 (W_f) and 1.0e-4 with the
    # small-batch kernels at the two seeds, 1.5e-4 and 3.0e-4 (W_r) with the general ones: which entries flip, not which kernel.
    assert worst[0][0] <= 1e-5
    assert worst[1][0] <= 4e-4
    g.close()
