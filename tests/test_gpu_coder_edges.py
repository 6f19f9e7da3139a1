"""The coder where one launch takes a stream through many steps: step counts around the four rows of tables it keeps in
flight, payloads shorter than the eight bytes the decoder reads at a time, streams that fill no workgroup, tables
with frequencies of 0, and a job whose pieces end inside the uniform warm-up. Integers: bit for bit against the oracle's coder, or the job in one piece."""
import os

import numpy as np
import pytest

import fade_inputs as fi
import oracle as orc
from gpu_helpers import make_pair, need_gpu


@pytest.mark.gpu
@pytest.mark.parametrize("n_streams,n_steps,conc", [(5, 1, 1.0), (1, 3, 0.02), (6, 4, 0.3), (3, 5, 0.02), (66, 7, 0.005), (2, 33, 0.002)])
def test_coder_under_tables_at_step_edges(n_streams, n_steps, conc):
    torch = need_gpu()
    g, _, _ = make_pair(4, 8, 32, 64, "bf16")
    rng = np.random.default_rng(100 * n_streams + n_steps)
    f = orc.quantize(rng.dirichlet(np.full(256, conc), n_steps * n_streams).astype(np.float32)).reshape(n_steps, n_streams, 256)
    sym = (np.cumsum(f.astype(np.int64), 2) > rng.integers(0, 65536, (n_steps, n_streams, 1))).argmax(2).astype(np.uint8)
    sym[::3] = rng.choice(np.array([0, 3, 252, 255], np.uint8), sym[::3].shape)  # ends of a lane's four symbols, rare ones
    cap = 3 * n_steps + 3
    print(f"coder edges streams={n_streams} steps={n_steps}", flush=True)
    fd, sd = torch.from_numpy(f.view(np.int16)).cuda(), torch.from_numpy(sym).cuda()
    out = torch.full((n_streams, cap), 0xA5, dtype=torch.uint8, device="cuda")
    ln = torch.zeros(n_streams, dtype=torch.int32, device="cuda")
    g.coder_encode_tables(fd, sd, n_steps, n_streams, out, cap, ln)
    o, l = out.cpu().numpy(), ln.cpu().numpy()
    for k in range(n_streams):
        ref = orc.coder_encode(f[:, k], sym[:, k])
        assert l[k] == ref.size and o[k, :l[k]].tobytes() == ref.tobytes(), k
        assert (o[k, l[k]:] == 0xA5).all()
    back = torch.zeros((n_steps, n_streams), dtype=torch.uint8, device="cuda")
    g.coder_decode_tables(fd, n_steps, n_streams, out, cap, ln, back)
    np.testing.assert_array_equal(back.cpu().numpy(), sym)
    g.close()


def _dyadic_lines():
    out = []
    for line in open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "coder_dyadic.txt")):
        if line.strip() and not line.startswith("#"):
            out.append(np.array([int(s) for s in line.split(";")[0].split()], np.uint8))
    return out


def _zero_frequency_streams(n_steps):
    """(tables [n_steps][streams][256], symbols [n_steps][streams]): streams whose tables give some symbols, the last ones above
    all, the frequency 0. The interval is the full 2^32 at every stream's first symbol, and after every symbol of a dyadic table."""
    rng = np.random.default_rng(8)
    tabs, syms = [], []

    def add(rows, sym):
        tabs.append(np.broadcast_to(rows, (n_steps, 256)).astype(np.uint16))
        syms.append(np.resize(np.asarray(sym, np.uint8), n_steps))

    dyadic = np.zeros(256, np.int64)
    dyadic[:4] = [32768, 16384, 8192, 8192]
    for line in _dyadic_lines():
        add(dyadic, line)
    for used in (2, 3, 5, 6, 7, 8, 27, 250, 251, 253, 254):  # every place of the last used symbol among a lane's four
        f = np.zeros(256, np.int64)
        f[:used] = rng.multinomial(65536 - used, rng.dirichlet(np.ones(used))) + 1
        add(f, rng.integers(0, used, n_steps))
        add(f, np.full(n_steps, used - 1))
        halves = np.zeros(256, np.int64)  # powers of two down to two equal last ones
        k = min(used, 15)
        halves[used - k:used] = [1 << (15 - i) for i in range(k - 1)] + [1 << (17 - k)]
        add(halves, rng.integers(used - k, used, n_steps))
    holes = np.zeros((n_steps, 256), np.int64)  # frequency 0 anywhere, another table at every step
    sym = np.zeros(n_steps, np.uint8)
    for i in range(n_steps):
        live = np.sort(rng.choice(256, 40, replace=False))
        holes[i, live] = rng.multinomial(65536 - 40, rng.dirichlet(np.full(40, 0.2))) + 1
        sym[i] = rng.choice(live)
    add(holes, sym)
    return np.stack(tabs, 1), np.stack(syms, 1)


def test_zero_frequency_fixture_round_trips_in_the_oracle():
    f, sym = _zero_frequency_streams(21)
    assert (f.astype(np.int64).sum(2) == 65536).all()
    for k in range(f.shape[1]):
        np.testing.assert_array_equal(orc.coder_decode(f[:, k], len(f), orc.coder_encode(f[:, k], sym[:, k])), sym[:, k])


@pytest.mark.gpu
def test_coder_under_tables_with_zero_frequencies():
    torch = need_gpu()
    g, _, _ = make_pair(4, 8, 32, 64, "bf16")
    n_steps = 21
    f, sym = _zero_frequency_streams(n_steps)
    n_streams, cap = f.shape[1], 4 * n_steps + 4
    print(f"coder, tables with zeros: streams={n_streams}", flush=True)
    fd, sd = torch.from_numpy(f.view(np.int16)).cuda(), torch.from_numpy(sym).cuda()
    out = torch.zeros((n_streams, cap), dtype=torch.uint8, device="cuda")
    ln = torch.zeros(n_streams, dtype=torch.int32, device="cuda")
    g.coder_encode_tables(fd, sd, n_steps, n_streams, out, cap, ln)
    o, l = out.cpu().numpy(), ln.cpu().numpy()
    for k in range(n_streams):
        assert o[k, :l[k]].tobytes() == orc.coder_encode(f[:, k], sym[:, k]).tobytes(), k
    back = torch.zeros((n_steps, n_streams), dtype=torch.uint8, device="cuda")
    g.coder_decode_tables(fd, n_steps, n_streams, out, cap, ln, back)
    np.testing.assert_array_equal(back.cpu().numpy(), sym)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("cuts", [(1,), (3, 8), (7, 9)])
def test_pieces_that_end_inside_the_uniform_warm_up(cuts):
    torch = need_gpu()
    import paper_2604_07239_amd as fa
    B, T, n = 7, 8, 7 * 24 - 5  # the last stream is short
    g = fa.Fade(fa.make_config(B, T, 32, 64, dtype=fa.BF16))
    g.load_weights(fi.init_blob(B, T, 32, 64, 3).data)
    src = torch.from_numpy(fi.text(9, n)).cuda()
    g.encode_device(src, n)
    lens, data = g.payloads()
    at = 0
    for c in cuts + (0,):
        g.encode_device(src, n, at, c - at if c else 0)
        at = c
    lens2, data2 = g.payloads()
    np.testing.assert_array_equal(lens2, lens)
    assert data2.tobytes() == data.tobytes()
    dst = torch.zeros(n, dtype=torch.uint8, device="cuda")
    at = 0
    for c in cuts + (0,):
        g.decode_device(lens, data, dst, n, at, c - at if c else 0)
        at = c
    assert torch.equal(dst, src)
    g.close()
