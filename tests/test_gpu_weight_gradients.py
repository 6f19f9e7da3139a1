"""The launch that shares all 256 x 256 weight-gradient tiles out in equal pieces, at batches that end inside a block of 64 rows:
gradients of one step against the oracle, an active stream in every block (the others have a gradient of zero), so that a block that is
left out, taken twice or read from another place shows wherever a workgroup's share or a range of the batch ends."""
import numpy as np
import pytest

import fade_inputs as fi
import oracle as orc
from gpu_helpers import need_gpu
from test_gpu_online import _compare_gradients, _sub_view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,H,widths,launch", [
    (2050, 64, 512, {}, True),    # 192 tiles of 33 blocks, one range: the smallest batch that takes the launch
    (2170, 64, 512, {}, True),    # 34 blocks: two ranges of 17, shares that end inside them
    (8200, 32, 320, {}, True),    # 32 tiles of 129 blocks (gradients of W_c, W_r): eight workgroups to a tile
    (8300, 32, 320, {}, True),    # 130 blocks: two ranges, four workgroups to each
    (8192, 32, 320, {}, True),    # 128 blocks: 16 ranges, a workgroup's share is two of them
    (8192, 16, 64, dict(d_cache=64, d_e=1024), True),    # one matrix of 16 tiles (W_fg | W_fv): 16 ranges give every compute unit one
    (2111, 16, 64, dict(d_cache=4096, d_e=8192), True),  # 224 tiles of a wide refiner, one row short of a block
    (4096, 16, 64, dict(d_cache=512, d_e=8192), True),   # gradient at H_coarse: 32 tiles x 8 ranges of its own on 256 x 256
    (4096, 8, 64, dict(d_cache=512, d_e=8192), False)])  # the same with 16 tiles x 16 ranges of 1024, the most ranges
def test_weight_gradients_of_ragged_batches(B, T, H, widths, launch, monkeypatch):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    D = 32
    blocks = np.arange((B + 63) // 64)
    idx = np.unique(np.r_[0, np.minimum(64 * blocks + 37 * blocks % 64, B - 1), B - 2, B - 1])  # 37: the rows wander through the blocks
    act = np.zeros(B, np.uint8)
    act[idx] = 1
    blob = fi.init_blob(B, T, D, H, 7, std=0.05, **widths)
    monkeypatch.setenv("FADE_DEBUG_WU_GRAD", "1")  # the sums of the slices go to the gradient array
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, update_mode=fa.ONLINE_ADAM, **widths))
    g.load_weights(blob.data)
    sub = fi.Blob(len(idx), T, D, H, **widths)
    for name, _, _ in sub.specs:
        sub[name] = blob[name][idx] if name == "W_U" else blob[name]
    o = orc.Oracle(orc.make_config(len(idx), T, D, H, dtype=orc.BF16, update_mode=orc.ONLINE_ADAM, **widths))
    o.load_weights(sub.data)
    data = np.random.default_rng(B).integers(0, 256, (B, T + 1), dtype=np.uint8)
    win, tgt = np.ascontiguousarray(data[:, :T]), np.ascontiguousarray(data[:, T])
    ad = torch.from_numpy(act).cuda()
    g.profile(True)
    g.step_probs(torch.from_numpy(win).cuda(), ad, None, None)
    o.step_probs(np.ascontiguousarray(win[idx]), None)
    go = o.backward(np.ascontiguousarray(tgt[idx]), None)
    g.step_update(torch.from_numpy(tgt).cuda(), ad)
    assert ("gemms_weights" in g.profile_read()) == launch
    _compare_gradients(sub, _sub_view(blob, sub, g.debug_grad(), idx), go, 3e-2, f"B={B}")
    g.close()


@pytest.mark.parametrize("B,T,H,matrices,bar", [
    # sums over at most 2048 rows are exact: a product of two bf16 has 16 significant bits, 128 k-steps of 16 equal rows add 7
    (4096, 64, 512, ("W_m", "W_r", "W_c", "W_fg", "W_fv", "W_f"), 1e-12),
    (16384, 32, 512, ("W_r", "W_c", "W_fg", "W_fv"), 1e-12),
    # 4096 rows in one chain, 256 k-steps of equal terms: below 2 ** k half the steps err by at most half a unit of 2 ** (k - 24), the
    # binades below by a quarter of that each time: 256 / 3 units of 2 ** -24 of the sum
    (16384, 64, 512, ("W_m", "W_r", "W_c", "W_fg", "W_fv", "W_f"), 256 / 3 * 2.0 ** -24)])
def test_sums_over_many_rows_do_not_drift(B, T, H, matrices, bar, monkeypatch):
    """Every stream the same: a weight gradient is then B times the outer product of two bf16 vectors, and what its best approximation
    by one outer product (in 64 bits) leaves of it is the rounding of the sums, which grows with the rows added in one chain."""
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    D = 32
    monkeypatch.setenv("FADE_DEBUG_WU_GRAD", "1")  # the sums of the slices go to the gradient array
    one, blob = fi.init_blob(1, T, D, H, 7, std=0.05), fi.Blob(B, T, D, H)
    for name, _, _ in one.specs:
        blob[name] = np.broadcast_to(one[name], blob[name].shape) if name == "W_U" else one[name]
    g = fa.Fade(fa.make_config(B, T, D, H, dtype=fa.BF16, update_mode=fa.ONLINE_ADAM))
    g.load_weights(blob.data)
    g.step_probs(torch.from_numpy(np.tile(fi.text(3, T), (B, 1))).cuda(), None, None, None)
    g.step_update(torch.full((B,), 101, dtype=torch.uint8, device="cuda"))
    blob.data[:] = np.asarray(g.debug_grad()).reshape(-1)
    g.close()
    for name in matrices:
        G = torch.from_numpy(blob[name].astype(np.float64)).cuda()
        right = G[G.norm(dim=1).argmax()].clone()
        for _ in range(3):  # power iteration on what is one outer product but for rounding
            right /= right.norm()
            left = G @ right
            right = G.t() @ left
        right /= right.norm()
        rest = G - (G @ right)[:, None] * right[None, :]
        assert float(rest.norm() / G.norm()) <= bar, name
