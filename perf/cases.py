"""The work that users of the codec have it do, as cases that can be timed.

A case names one call sequence of the public binding on one batch of intermediate features: the direction
(encode, decode, or one after the other), the element type, the shape (rows = codec instances), the kind of
values, and the codec's options.  Shapes and options are those of the five workloads of
paper_2511_11608_amd/synth.py and of bench.py, plus what lies between and around them: one client instead of
256, rows whose length is no multiple of anything, asymmetric thresholds, a fixed ladder, the mismatch guard,
two-dimensional instances.
"""
import math

import torch

from paper_2511_11608_amd import binding
from paper_2511_11608_amd.synth import BITS_2_TO_8

LARGEST_BYTES = 16384 * 4096 * 2        # input of the largest case: 16384 tokens of 4096 bf16 values
RAGGED_ELEMENTS = 2048 * 3001           # input of the ragged case


def _case(name, op, dtype, rows, row_len, values, keep, blocks, mode="budget", level=1e-3, n_cols=0, header=False):
    """level: the budget (modes budget, csr), delta (ds) or lambda (atkf; its budget is 1e-3); unused by ladder."""
    c = {"op": op, "dtype": dtype, "rows": rows, "row_len": row_len, "values": values, "keep": keep, "blocks": blocks,
         "mode": mode, "level": level, "n_cols": n_cols, "header": header}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one client sends the hidden state of one decoding step, in the paper's fixed multi-level mode: pure latency
        _case("client_step_encode", "encode", "bf16", 1, 4096, "hidden", 0.10, 8, "ladder"),
        # one auto-regressive decoding step of 256 clients, and the server's side of it
        _case("ar_step_encode", "encode", "bf16", 256, 8192, "hidden", 0.10, 8),
        _case("ar_step_decode", "decode", "bf16", 256, 8192, "hidden", 0.10, 8),
        # one post-ReLU CNN feature map as a single instance; the receiver learns the shape from the header
        _case("map_encode", "encode", "f32", 1, 200704, "relu", 0.10, 4),
        _case("map_decode_header", "decode", "f32", 1, 200704, "relu", 0.10, 4, header=True),
        # a batch of CNN feature maps, flat and as channels x positions with CSR blocks (both directions)
        _case("batch_encode", "encode", "f32", 32, 401408, "channels", 0.20, 16, n_cols=784),
        _case("batch_csr", "both", "f32", 32, 401408, "channels", 0.20, 16, "csr", n_cols=784),
        # vision-transformer tokens, with the plain and the asymmetric thresholds (outlier channels of one sign)
        _case("tokens_encode", "encode", "f32", 12608, 768, "tokens", 0.15, 8, level=5e-4),
        _case("tokens_encode_atkf", "encode", "f32", 12608, 768, "tokens", 0.15, 8, "atkf", 0.1),
        # the hidden states of a prefill: the largest batch, both directions
        _case("prefill_encode", "encode", "bf16", 16384, 4096, "hidden", 0.10, 8),
        _case("prefill_decode", "decode", "bf16", 16384, 4096, "hidden", 0.10, 8),
        # rows of odd length (a pruned width): no row starts where the one before it did, modulo 16 bytes
        _case("ragged_both", "both", "bf16", 2048, 3001, "hidden", 0.10, 8),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pick(rng, weighted):
    names, weights = zip(*weighted)
    return rng.choices(names, weights)[0]


def draw(rng):
    op = _pick(rng, [("encode", 3), ("decode", 2)])
    blocks = rng.choice([4, 8, 16])
    n_cols = 0
    if rng.random() < 0.7:              # token rows: hidden widths, padded ones, and any width
        width = _log_uniform(rng, 256, 12288)
        kind = _pick(rng, [(64, 6), (8, 2), (1, 2)])
        width = width // 64 * 64 if kind == 64 else width // 8 * 8 if kind == 8 else width | 1
        dtype = _pick(rng, [("bf16", 2), ("f32", 1)])
        most = LARGEST_BYTES // (width * (2 if dtype == "bf16" else 4))
        if kind == 1:
            most = min(most, RAGGED_ELEMENTS // width)
        rows = min(_log_uniform(rng, 1, 16384), most)
        values = "hidden" if dtype == "bf16" else "tokens"
        mode = _pick(rng, [("budget", 12), ("ladder", 3), ("ds", 2), ("atkf", 3)])
        keep = rng.choice([0.05, 0.10, 0.15, 0.20, 0.25])
    else:                               # feature maps: channels x positions, a few per batch
        while True:
            channels, side = _log_uniform(rng, 32, 512), rng.randint(7, 56)
            if rng.random() < 0.8:
                channels = channels // 8 * 8
            if channels * side * side <= 401408:
                break
        n_cols, width = side * side, channels * side * side
        rows = _log_uniform(rng, 1, 32)
        if width % 8:
            rows = max(1, min(rows, RAGGED_ELEMENTS // width))
        dtype = _pick(rng, [("f32", 3), ("bf16", 1)])
        values = _pick(rng, [("relu", 1), ("channels", 1)])
        mode = _pick(rng, [("budget", 3), ("ladder", 1), ("csr", 1)])
        keep = rng.choice([0.05, 0.10, 0.15, 0.20])
    if keep * width < 4 * blocks:
        blocks = 4
    level = {"budget": rng.choice([5e-4, 1e-3, 2e-3]), "csr": 1e-3, "ds": 0.3, "atkf": 0.1, "ladder": 0.0}[mode]
    return _case(None, op, dtype, rows, width, values, keep, blocks, mode, level, n_cols,
                 header=op == "decode" and rng.random() < 0.25)


def _values(case, seed):
    """The synthetic features of paper_2511_11608_amd/synth.py, drawn on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    R, N, kind = case["rows"], case["row_len"], case["values"]
    out = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    x = torch.empty((R, N), device="cuda").normal_(generator=g)

    def uniform(*shape):
        return torch.empty(shape, device="cuda").uniform_(generator=g)

    def channels_of(n):
        return torch.randperm(N, generator=g, device="cuda")[:n]

    if kind == "hidden":                # normal with Laplace tails, 0.1 % of the channels are outliers
        x *= 0.5
        pick = uniform(R, N) < 0.1
        u = uniform(R, N) - 0.5
        lap = -0.5 * torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999))
        x = torch.where(pick, lap, x)
        x[:, channels_of(max(1, round(0.001 * N)))] *= 50.0
    elif kind == "tokens":              # normal, two outlier channels
        x[:, channels_of(2)] *= 30.0
    elif kind == "relu":                # half exact zeros, the rest half-normal
        x = x.abs_() * (uniform(R, N) < 0.5)
    else:                               # 60 % zeros, the rest half-normal at the channel's scale
        cols = case["n_cols"]
        sigma = 0.2 + 1.8 * uniform(N // cols)
        x = x.abs_() * (uniform(R, N) < 0.4) * sigma.repeat_interleave(cols)
    return x.to(out).contiguous()


def _ladder(blocks):
    return [max(2, 8 - m * 8 // blocks) for m in range(blocks)]


def _encode(s):
    c, bufs = s["case"], s["bufs"]
    if c["mode"] == "ladder":
        binding.slicer_encode_ladder(s["x"], c["keep"], s["ladder"], *bufs)
    elif c["mode"] == "ds":
        binding.slicer_encode_ds(s["x"], c["keep"], c["blocks"], BITS_2_TO_8, c["level"], *bufs)
    elif c["mode"] == "atkf":
        binding.slicer_encode_atkf(s["x"], c["keep"], c["level"], c["blocks"], c["blocks"], BITS_2_TO_8, 1e-3, *bufs)
    elif c["mode"] == "csr":
        binding.slicer_encode_csr(s["x"], c["row_len"] // c["n_cols"], c["n_cols"], c["keep"], c["blocks"], BITS_2_TO_8,
                                  c["level"], *bufs)
    else:
        binding.slicer_encode(s["x"], c["keep"], c["blocks"], BITS_2_TO_8, c["level"], *bufs)


def _decode(s):
    c, (stream, meta, _) = s["case"], s["bufs"]
    if c["header"]:
        binding.slicer_decode(stream, meta, s["y"])
    elif c["mode"] == "csr":
        binding.slicer_decode_as_csr(stream, meta, s["y"], c["row_len"] // c["n_cols"], c["n_cols"], c["blocks"])
    else:
        binding.slicer_decode_as(stream, meta, s["y"], c["blocks"])


def prepare(case, seed):
    """Encoder: features and the call's buffers.  Decoder: a received stream and its meta, and the output tensor."""
    s = {"case": case, "x": _values(case, seed), "ladder": _ladder(case["blocks"])}
    bits = binding.slicer_ladder_bit_set(s["ladder"]) if case["mode"] == "ladder" else BITS_2_TO_8
    if case["mode"] == "csr":
        s["bufs"] = binding.alloc_buffers_csr(s["x"], case["row_len"] // case["n_cols"], case["n_cols"], case["keep"],
                                              case["blocks"], bits)
    else:
        s["bufs"] = binding.alloc_buffers(s["x"], case["keep"], case["blocks"], bits)
    s["bufs"][0].zero_()                # the words behind the stream's end stay as they are: zeros
    if case["op"] != "encode":
        s["y"] = torch.empty_like(s["x"])
    if case["op"] == "decode":
        _encode(s)
        s["x"], s["bufs"] = None, (s["bufs"][0], s["bufs"][1], None)
    return s


def run(s):
    op = s["case"]["op"]
    if op != "decode":
        _encode(s)
    if op != "encode":
        _decode(s)
    if op == "decode":
        return s["y"]
    return s["bufs"][:2] if op == "encode" else (*s["bufs"][:2], s["y"])


def work(case):
    R, N, M = case["rows"], case["row_len"], case["blocks"]
    k = int(case["keep"] * N)
    dense = R * N * (2 if case["dtype"] == "bf16" else 4)
    bits = {"ladder": sum(_ladder(M)) / M, "ds": 8.0}.get(case["mode"], 5.0)      # of a code, about
    if case["mode"] == "csr":
        index = k * math.ceil(math.log2(case["n_cols"])) + 2 * M * (N // case["n_cols"] + 1) * math.ceil(math.log2(k + 1))
    else:
        index = k * math.ceil(math.log2(N))
    coded = R * (index + k * bits) / 8 + 64 + 16 * R + 18 * R * M
    # per sent value: offset, scale, round and the reconstruction; the search does about as much for every bitwidth
    ops = R * k * {"encode": 4 + (0 if case["mode"] == "ladder" else 4 * 7), "decode": 2, "both": 6 + 4 * 7}[case["op"]]
    return {"bytes": (dense + coded) * (2 if case["op"] == "both" else 1), "flops": ops}


def tolerance(case):
    return "exact"                      # the format is bytes; the decoder's arithmetic is fixed to the last bit
