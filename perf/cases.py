"""The work that programs have this library do, as a list of measurable cases: single model steps, online adaptation,
compression jobs in both update modes and both operand types, whole containers on host buffers, and the stand-alone
integer kernels. Sizes are those of the benchmark configurations (`fade_inputs.CONFIGS`) or of the tests, plus ragged ones.

Kinds of case, each through the public calls of `paper_2604_07239_amd.Fade`:
  step       `steps` calls of step_probs in mid-stream (frozen weights): a program that evaluates or drives its own coder.
  adapt      reset, then `steps` times step_probs + step_update, then the adapted weights read out: a program that fits the
             model to a sample and keeps the result.
  job        a device-resident job, compressed (encode_device, payloads) and decompressed again (decode_device).
  container  the same from host buffers (encode, decode), with a length that is no multiple of the stream count.
  tables     quantize, coder_encode_tables, coder_decode_tables on given probabilities: a program with its own model.

The payload bytes of a job are no output of it here: the coder turns a table that differs in one entry into other bytes from
there on, and tables follow the last bit of the probabilities, so two correct implementations of the same precision share
hardly any. What they have to share is the decoded job, to the byte, and every stream's rate.
"""
import math

import numpy as np
import torch

import paper_2604_07239_amd as fade

D_LOW, TAPS = 64, 3


def listed():
    return [
        # one step of a handful of streams in fp32: the smallest call, launch latency and nothing else
        dict(name="step-f32-b16", kind="step", dtype="f32", B=16, T=32, D=16, H=128, steps=1, source="text"),
        # adaptation of that model, a few symbols at a time: the smallest backward pass
        dict(name="adapt-f32-b16", kind="adapt", dtype="f32", B=16, T=32, D=16, H=128, steps=8, source="text"),
        # benchmark configuration 1 as a job: 16 streams, fp32, weights updated after every symbol
        dict(name="job-f32-online-b16", kind="job", dtype="f32", B=16, T=32, D=16, H=128, steps=128, mode="online", source="text"),
        # one step at the stream count of configuration 2: latency of a decoder that serves many streams
        dict(name="step-bf16-b1024", kind="step", dtype="bf16", B=1024, T=64, D=32, H=256, steps=1, source="text"),
        # bf16 adaptation with a short window on a small batch
        dict(name="adapt-bf16-b128", kind="adapt", dtype="bf16", B=128, T=16, D=32, H=512, steps=4, source="text"),
        # configuration 2, inference only: compression takes many steps per pass, decompression one
        dict(name="job-frozen-b1024", kind="job", dtype="bf16", B=1024, T=64, D=32, H=256, steps=256, mode="frozen", source="text"),
        # configuration 2 as the method defines it
        dict(name="job-online-b1024", kind="job", dtype="bf16", B=1024, T=64, D=32, H=256, steps=128, mode="online", source="text"),
        # configuration 5, inference only: the largest batch, where both directions take single steps
        dict(name="job-frozen-b16384", kind="job", dtype="bf16", B=16384, T=64, D=32, H=512, steps=64, mode="frozen", source="float"),
        # configuration 5 as the method defines it: the headline workload
        dict(name="job-online-b16384", kind="job", dtype="bf16", B=16384, T=64, D=32, H=512, steps=64, mode="online", source="float"),
        # the paper's default model shape (configuration 6): a short window under a wide cache and a wide refiner
        dict(name="job-online-wide-b4096", kind="job", dtype="bf16", B=4096, T=16, D=32, H=8192, d_cache=4096, d_e=8192, steps=64,
             mode="online", source="text"),
        # a file of no round size from host memory, a stream count that fills no tile, a slot of six elements
        dict(name="container-online-b1500", kind="container", dtype="bf16", B=1500, T=32, D=32, H=192, steps=64, short=1237, mode="online",
             source="genome"),
        # a model elsewhere, only its tables and the coder here
        dict(name="tables-b4096", kind="tables", streams=4096, steps=32),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["step", "adapt", "job", "job", "job", "container", "tables"])
    if kind == "tables":
        streams = _log_int(rng, 16, 16384)
        return dict(kind=kind, streams=streams, steps=max(4, min(64, (1 << 17) // streams)))
    source = rng.choice(["text", "genome", "float"])
    if rng.random() < 0.25:  # the fp32 path serves small batches
        c = dict(kind=kind, dtype="f32", B=_log_int(rng, 4, 64), T=32, D=16, H=rng.choice([128, 256]), source=source)
    else:
        high = 1024 if kind == "adapt" else 16384
        c = dict(kind=kind, dtype="bf16", B=_log_int(rng, 32, high), T=rng.choice([16, 32, 64]), D=32, H=rng.choice([128, 192, 256, 384, 512]),
                 source=source)
    if kind == "step":
        c["steps"] = rng.choice([1, 2, 4])
    elif kind == "adapt":
        c["steps"] = rng.choice([2, 3, 4])
    else:
        c["mode"] = rng.choice(["online", "online", "frozen"])
        c["steps"] = min(_log_int(rng, 24, 160), (1 << 20) // c["B"])
        if kind == "container":
            c["short"] = rng.randrange(1, c["T"] + c["steps"]) if c["B"] < 64 else rng.randrange(1, c["B"])
    return c


def _widths(case):
    dc, de = case.get("d_cache", case["H"]), case.get("d_e", case["H"])
    return dc, de, dc // case["T"]


def _bytes_of(source, seed, n):
    """n bytes with the statistics of a text, a genome or a series of 32-bit floats."""
    r = np.random.default_rng(seed)
    if source == "genome":
        out = r.choice(np.frombuffer(b"ACGT", np.uint8), n, p=[0.3, 0.2, 0.2, 0.3])
        out[r.random(n) < 0.01] = ord("N")
        return out
    if source == "float":
        walk = np.cumsum(r.standard_normal(n // 4 + 1)).astype(np.float32)
        return walk.view(np.uint8)[:n].copy()
    lengths = r.integers(1, 9, 2048)
    letters = np.frombuffer(b"etaoinshrdlcumwfgypbvkxjqz", np.uint8)
    pick = np.minimum(r.geometric(0.12, int(lengths.sum())) - 1, letters.size - 1)
    words = np.split(letters[pick], np.cumsum(lengths)[:-1])
    words = [w.tobytes() + b" " for w in words]
    rank = np.minimum(r.zipf(1.3, n // 2 + 1) - 1, len(words) - 1)
    return np.frombuffer(b"".join([words[k] for k in rank]), np.uint8)[:n].copy()


def _weights(case, seed):
    """The canonical blob at random initialisation: matrices N(0, 0.02), gains and residual scales 1, shifts and biases 0."""
    B, T, D = case["B"], case["T"], case["D"]
    dc, de, c = _widths(case)
    dh = T * D
    tensors = [(256 * D, None), (D, 1), (D, 0), (D, 1), (D, 0), (D * c, None), (D * c, None), (dc * dh, None), (1, 1), (TAPS * D * D, None),
               (D, 0), (dh * dh, None), (dh, 1), (dh, 0), (dh * D_LOW, None), (B * D_LOW * D_LOW, None), (D_LOW * dh, None), (dh * dh, None),
               (1, 1), (dh, 1), (dh, 0), (dh * de, None), (dh * de, None), (de * dh, None), (dh, 1), (dh, 0), (1, 1), (dh * 256, None), (256, 0)]
    blob = torch.empty(sum(n for n, _ in tensors), device="cuda")
    blob.normal_(0.0, 0.02, generator=torch.Generator(device="cuda").manual_seed(seed))
    at = 0
    for n, fill in tensors:
        if fill is not None:
            blob[at:at + n] = fill
        at += n
    return blob.cpu().numpy()


def _context(case, seed, online):
    ctx = fade.Fade(fade.make_config(case["B"], case["T"], case["D"], case["H"], d_cache=case.get("d_cache", 0), d_e=case.get("d_e", 0),
                                     dtype=fade.BF16 if case["dtype"] == "bf16" else fade.F32,
                                     update_mode=fade.ONLINE_ADAM if online else fade.FROZEN))
    ctx.load_weights(_weights(case, seed))
    return ctx


def prepare(case, seed):
    kind = case["kind"]
    if kind == "tables":
        rows = case["steps"] * case["streams"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        probs = torch.softmax(2.0 * torch.randn((rows, 256), device="cuda", generator=g), dim=1)
        shape = (case["steps"], case["streams"])
        cap = 4 * case["steps"] + 16
        state = dict(probs=probs, sym=torch.multinomial(probs, 1, generator=g).to(torch.uint8).reshape(shape),
                     freq=torch.zeros((*shape, 256), dtype=torch.int16, device="cuda"), cap=cap,
                     out=torch.zeros((case["streams"], cap), dtype=torch.uint8, device="cuda"),
                     len=torch.zeros(case["streams"], dtype=torch.int32, device="cuda"),
                     back=torch.zeros(shape, dtype=torch.uint8, device="cuda"),
                     ctx=fade.Fade(fade.make_config(16, 32, 32, 128)))  # these calls need a context, and no weights
        torch.cuda.synchronize()
        return dict(case=case, **state)
    B, T, steps = case["B"], case["T"], case["steps"]
    state = dict(case=case, ctx=_context(case, seed, kind == "adapt" or case.get("mode") == "online"))
    if kind in ("step", "adapt"):
        lead = T if kind == "step" else 0  # a step is measured in mid-stream: the rolling cache holds the T steps before
        text = torch.from_numpy(_bytes_of(case["source"], seed, B * (T + lead + steps)).reshape(B, -1)).cuda()
        windows = text.unfold(1, T, 1).permute(1, 0, 2).contiguous()  # [step][stream][T]
        state["targets"] = text[:, T:].t().contiguous()
        state["probs"] = torch.zeros((steps, B, 256), device="cuda")
        torch.cuda.synchronize()
        for i in range(lead):
            state["ctx"].step_probs(windows[i])
        state["windows"] = windows[lead:].contiguous()
    elif kind == "job":
        state["n"] = B * (T + steps)
        state["src"] = torch.from_numpy(_bytes_of(case["source"], seed, state["n"])).cuda()
        state["dst"] = torch.zeros(state["n"], dtype=torch.uint8, device="cuda")
    else:
        state["src"] = _bytes_of(case["source"], seed, B * (T + steps) - case["short"])
    torch.cuda.synchronize()
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "step":
        for i in range(case["steps"]):
            ctx.step_probs(state["windows"][i], None, None, state["probs"][i])
        return state["probs"]
    if kind == "adapt":
        ctx.reset()
        for i in range(case["steps"]):
            ctx.step_probs(state["windows"][i], None, None, state["probs"][i])
            ctx.step_update(state["targets"][i])
        return {"probs": state["probs"], "weights": ctx.get_weights()}
    if kind == "tables":
        streams, steps, cap = case["streams"], case["steps"], state["cap"]
        ctx.quantize(state["probs"], state["freq"])
        ctx.coder_encode_tables(state["freq"], state["sym"], steps, streams, state["out"], cap, state["len"])
        ctx.coder_decode_tables(state["freq"], steps, streams, state["out"], cap, state["len"], state["back"])
        return {"freq": state["freq"], "payload": state["out"], "lengths": state["len"], "symbols": state["back"]}
    if kind == "job":
        n = state["n"]
        ctx.encode_device(state["src"], n)
        lengths, payload = ctx.payloads()
        ctx.decode_device(lengths, payload, state["dst"], n)
        decoded = state["dst"]
    else:
        blob = ctx.encode(state["src"])
        decoded = ctx.decode(blob, state["src"].size)
        lengths = blob[64:64 + 4 * case["B"]].view(np.uint32)
    return {"decoded": decoded, "bits_per_byte": lengths * np.float32(8.0 / (case["T"] + case["steps"]))}


def work(case):
    if case["kind"] == "tables":
        # per row: probabilities read once, the table written once and read by each direction of the coder; a few integer
        # operations per entry
        rows = case["steps"] * case["streams"]
        return {"bytes": rows * (4 * 256 + 3 * 2 * 256), "flops": rows * 4 * 256}
    B, T, D, steps = case["B"], case["T"], case["D"], case["steps"]
    dc, de, c = _widths(case)
    dh = T * D
    element = 2 if case["dtype"] == "bf16" else 4
    shared = dc * dh + 2 * dh * dh + 2 * D_LOW * dh + 3 * de * dh + 256 * dh + 2 * D * c + TAPS * D * D + 256 * D
    memory = B * D_LOW * D_LOW
    forward = 2 * B * (2 * D * c + dc * dh + T * TAPS * D * D + 2 * dh * dh + 2 * dh * D_LOW + D_LOW * D_LOW + 3 * de * dh + 256 * dh)
    online = case["kind"] == "adapt" or case.get("mode") == "online"
    directions = 2 if case["kind"] in ("job", "container") else 1
    # forward: cache row and window per stream and step; an update takes two more products per forward one and
    # reads and writes weight and both moments of every parameter in fp32; frozen weights are read once per direction
    per_step = B * (T + 2 * dc * element)
    flops = forward
    if online:
        per_step += 24 * (shared + memory)
        flops = 3 * forward
    read = element * (shared + memory)
    if case["kind"] in ("step", "adapt"):
        read += 4 * 256 * B * steps
    if case["kind"] == "adapt":
        read += 4 * (shared + memory)
    return {"bytes": directions * (read + steps * per_step), "flops": directions * steps * flops}


def tolerance(case):
    """About four times what the path shows against the oracle, which computes in 64 bits on the same rounded weights."""
    if case["kind"] == "tables":
        return "exact"  # integers of given floats
    online = case["kind"] == "adapt" or case.get("mode") == "online"
    if case["kind"] == "step":  # probabilities: fp32 1.1e-7 (largest 5e-7), bf16 3.6e-3 (1.4e-2)
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 1.2e-2, "max": 6e-2}
    if case["kind"] == "adapt":
        # fp32: probabilities 4.3e-6, weights 1.3e-6 (largest 1.1e-3). bf16: 6.0e-3 and 2.5e-3 (0.14: an entry whose gradient
        # is within the error of zero may take Adam's first step of one learning rate the other way)
        return {"rel": 2e-5, "max": 5e-3} if case["dtype"] == "f32" else {"rel": 2e-2, "max": 0.5}
    # rates of whole bytes per stream: frozen 1.7e-3 (largest 6.9e-3), online 3.6e-3 (1.4e-2) in fp32 and 7.9e-3 (2.8e-2) in bf16;
    # one byte more or less is up to 2e-2 of a short stream that compresses well
    if not online:
        return {"rel": 7e-3, "max": 5e-2}
    return {"rel": 1.5e-2, "max": 6e-2} if case["dtype"] == "f32" else {"rel": 3e-2, "max": 0.12}
