"""Performance cases of the library: the calls that programs built on it make, over the sizes they make them at.

Five kinds of work, each through the package's public functions:

  step        one pass over `calls` equal-shaped layers of a network, Y_i = W_i X_i (`spmm`), captured once in a HIP graph
              and replayed: how a serving program runs calls of 5 to 20 us each, whose launches the host cannot keep up with
  spmm        one product called directly
  decode      one encrypted matrix decoded to bit planes, fp32 or bf16 (`decode`)
  encode      one matrix encrypted with Algorithm 1 (`encode`)
  exhaustive  the same with the search for the fewest patches (`encode_exhaustive`)

Weights are Gaussian draws, pruned by magnitude to the rate S, coded greedily into q bit planes with one scale per row and
plane, and encrypted on the GPU: the recipe of `synth_inputs`, made here with torch on the GPU so that a state takes
milliseconds.  X is Gaussian.  Shapes, rates and widths of the listed cases are those of `synth_inputs.CONFIGS`, of bench.py
and of the tests.
"""
import math

import numpy as np
import torch

import paper_1905_10138_amd as xe

DEV = "cuda:0"
KINDS = {"planes": xe.OUT_PLANES, "f32": xe.OUT_F32, "bf16": xe.OUT_BF16}


def _case(op, m, n, q, S, n_in, n_out=64, **more):
    c = {"op": op, "m": m, "n": n, "q": q, "S": S, "n_in": n_in, "n_out": n_out}
    c.update(more)
    return c


def listed():
    """The calls the listed cases stand for:

    tiny_f32_b8        the smallest direct call: a 256 x 256 layer and fp32 activations; host call and launch latency
    fig1_b64           the 2048 x 2048 layer and 64 columns of the paper's Fig. 1, a step over eight of them
    fc6_b1             one sample through fully-connected layers of 4096 x 9216 with two planes
    lstm_b32           gate matrices of 6000 x 3000 with three planes and a batch of 32 (3000 columns: a ragged last slice)
    large_b8           a large layer and few columns: the compressed bytes are what has to move
    fc6_b64            fully-connected layers, two planes, an ordinary batch
    large_b1024        the largest product: many columns, one plane
    wide_q2_b250       slices of 192 bits from 20 (the paper's preferred region), two planes, 250 columns stored without
                       padding, so that rows of X do not start on 16-byte boundaries
    fc6_f32_b64        fp32 activations at an ordinary size
    decode_bf16        a large matrix expanded to dense bf16 weights
    encode_q2          Algorithm 1 on a large two-plane matrix
    exhaustive_192_20  the search for the fewest patches at 2^20 inputs per slice, the offline step that takes longest
    """
    return [
        _case("spmm", 256, 256, 1, 0.90, 16, B=8, x="f32", pad=0, name="tiny_f32_b8"),
        _case("step", 2048, 2048, 1, 0.91, 16, B=64, x="bf16", pad=0, calls=8, name="fig1_b64"),
        _case("step", 4096, 9216, 2, 0.91, 16, B=1, x="bf16", pad=0, calls=8, name="fc6_b1"),
        _case("step", 6000, 3000, 3, 0.80, 24, B=32, x="bf16", pad=0, calls=8, name="lstm_b32"),
        _case("step", 16384, 4096, 1, 0.95, 8, B=8, x="bf16", pad=0, calls=8, name="large_b8"),
        _case("step", 4096, 9216, 2, 0.91, 16, B=64, x="bf16", pad=0, calls=8, name="fc6_b64"),
        _case("spmm", 16384, 4096, 1, 0.95, 8, B=1024, x="bf16", pad=0, name="large_b1024"),
        _case("spmm", 16384, 4096, 2, 0.95, 20, n_out=192, B=250, x="bf16", pad=0, name="wide_q2_b250"),
        _case("spmm", 4096, 9216, 2, 0.91, 16, B=64, x="f32", pad=0, name="fc6_f32_b64"),
        _case("decode", 16384, 4096, 2, 0.95, 8, kind="bf16", name="decode_bf16"),
        _case("encode", 16384, 4096, 2, 0.95, 8, name="encode_q2"),
        _case("exhaustive", 16384, 4096, 1, 0.95, 20, n_out=192, name="exhaustive_192_20"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: layers of 200 x 200 to 16384 x 9216, one to four planes, every slice width, any
    width of the encrypted vector that suits the pruning rate, 1 to 1024 columns, both types of X, padded and unpadded
    rows of X."""
    op = rng.choice(["spmm"] * 4 + ["step"] * 4 + ["decode"] * 2 + ["encode"] + ["exhaustive"])
    q = rng.choice([1, 1, 1, 2, 2, 3, 4])
    n_out = rng.choice([64, 64, 64, 128, 192, 256])
    S = rng.choice([0.80, 0.85, 0.90, 0.91, 0.95])
    # an encrypted vector holds at least about the mean number of kept weights of a slice
    low = min(30, max(4, math.ceil((1.0 - S) * n_out)))
    top = min(20 if op == "exhaustive" else 32, low + 16)
    low = min(low, top)
    n_in = rng.choice([k for k in (8, 16, 24) if low <= k <= top] or [top]) if rng.random() < 0.6 else rng.randint(low, top)
    m, n = _log_int(rng, 200, 16384), _log_int(rng, 200, 9216)
    if rng.random() < 0.5:  # half of the layers have round sizes
        m, n = max(256, m // 256 * 256), max(256, n // 256 * 256)
    n = min(n, max(200, 16384 * 4096 // m))
    if op == "decode":
        return _case(op, m, n, q, S, n_in, n_out=n_out, kind=rng.choice(["planes", "f32", "bf16"]))
    if op == "encode":
        return _case(op, m, n, q, S, n_in, n_out=n_out)
    if op == "exhaustive":  # network evaluations (dearer per weight for short slices) bounded by the listed case's
        while q * m * n * 2 ** n_in > 16384 * 4096 * 2 ** 20 * min(192, n_out) // 192:
            q, n_in = max(1, q - 1), n_in if q > 1 else n_in - 1
        return _case(op, m, n, q, S, n_in, n_out=n_out)
    x = rng.choice(["bf16", "bf16", "bf16", "f32"])
    pad = rng.choice([0, 0, 0, 1, 8])
    if op == "step":
        B = _log_int(rng, 1, 64)
        if rng.random() < 0.5 and B > 8:
            B = B // 8 * 8
        return _case(op, m, n, q, S, n_in, n_out=n_out, B=B, x=x, pad=pad, calls=rng.choice([4, 8]))
    most = 16384 * 4096 * 1024 // (m * n * q * (3 if x == "f32" else 1))
    B = _log_int(rng, 1, max(1, min(1024, most)))
    if rng.random() < 0.5 and B > 8:
        B = B // 8 * 8
    return _case(op, m, n, q, S, n_in, n_out=n_out, B=B, x=x, pad=pad)


# ---------------------------------------------------------------------------------------------- inputs

def _weights(case, seed):
    """Pruned, binary-coded weights: keep bool [m, n], planes bool [q, m, n], alpha fp32 [q, m] (GPU) and the rows of the
    XOR network (host uint32)."""
    m, n, q, S = case["m"], case["n"], case["q"], case["S"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    w = torch.randn((m, n), generator=g, device=DEV)
    keep = w.abs() > math.sqrt(2.0) * torch.erfinv(torch.tensor(S, dtype=torch.float64)).item()  # share S is pruned
    r = torch.where(keep, w, torch.zeros((), device=DEV))
    count = keep.sum(dim=1).clamp(min=1)
    planes, alpha = [], []
    for _ in range(q):
        a = r.abs().sum(dim=1) / count
        b = (r >= 0) & keep
        r = torch.where(keep, r - a[:, None] * torch.where(b, 1.0, -1.0), r)
        planes.append(b)
        alpha.append(a)
    bits = np.random.Generator(np.random.PCG64(seed)).integers(0, 2, size=(case["n_out"], case["n_in"]), dtype=np.uint64)
    M_rows = (bits << np.arange(case["n_in"], dtype=np.uint64)).sum(axis=1).astype(np.uint32)
    return keep, planes, torch.stack(alpha), M_rows


def _words(a, n_out):
    """xe.pack_bits on the GPU: bool [m, n] -> unit-major 64-bit words, rows padded to 32 and columns to n_out."""
    m, n = a.shape
    nrb, spr = -(-m // 32), -(-n // n_out) * (n_out // 64)
    p = torch.zeros((nrb * 32, spr * 64), dtype=torch.bool, device=a.device)
    p[:m, :n] = a
    p = p.view(nrb, 32, spr, 64).permute(0, 2, 1, 3)
    out = torch.zeros((nrb, spr, 32), dtype=torch.int64, device=a.device)
    for j in range(64):
        out |= p[..., j].to(torch.int64) << j
    return out.reshape(-1)


def _encoder_inputs(case, seed):
    keep, planes, alpha, M_rows = _weights(case, seed)
    return {"M_rows": M_rows, "mask": _words(keep, case["n_out"]),
            "planes": torch.stack([_words(b, case["n_out"]) for b in planes]), "alpha": alpha}


def _encode(case, e, fn):
    return fn(case["m"], case["n"], case["n_in"], case["q"], e["M_rows"], e["mask"], e["planes"], e["alpha"], n_out=case["n_out"])


def _layer_seed(seed, i):
    return seed * 64 + i


def _x(case, seed):
    """X of n x B values; `pad` more per row in memory (0: rows follow each other without a gap)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 7_000_000)
    dtype = torch.float32 if case["x"] == "f32" else torch.bfloat16
    buf = torch.randn((case["n"], case["B"] + case["pad"]), generator=g, device=DEV).to(dtype)
    return buf[:, :case["B"]]


def prepare(case, seed):
    op = case["op"]
    if op in ("encode", "exhaustive"):
        # the patch list's length is known only after the call: the program keeps it in an area that holds any list
        most = case["q"] * int(case["m"] * case["n"] * (1.0 - case["S"]) * 1.1 + 1000)
        return {"case": case, "inputs": _encoder_inputs(case, _layer_seed(seed, 0)),
                "patch": torch.zeros(most, dtype=torch.int16, device=DEV)}
    if op == "decode":
        layer = _encode(case, _encoder_inputs(case, _layer_seed(seed, 0)), xe.encode)
        return {"case": case, "layer": layer, "out": torch.empty_like(xe.decode(layer, KINDS[case["kind"]]))}
    layers, X, Y = [], [], []
    for i in range(case.get("calls", 1)):
        s = _layer_seed(seed, i)
        layers.append(_encode(case, _encoder_inputs(case, s), xe.encode))
        X.append(_x(case, s))
        Y.append(torch.empty((case["m"], case["B"]), dtype=torch.float32, device=DEV))
    state = {"case": case, "layers": layers, "X": X, "Y": Y}
    if op == "step":
        xe.spmm(layers[0], X[0], Y=Y[0])  # the library's first call on a device looks up its scratch memory
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for layer, x, y in zip(layers, X, Y):
                xe.spmm(layer, x, Y=y)
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "step":
        state["graph"].replay()
        return state["Y"]
    if op == "spmm":
        return xe.spmm(state["layers"][0], state["X"][0], Y=state["Y"][0])
    if op == "decode":
        return xe.decode(state["layer"], KINDS[case["kind"]], out=state["out"])
    layer = _encode(case, state["inputs"], xe.encode if op == "encode" else xe.encode_exhaustive)
    state["patch"][:layer.patch.numel()].copy_(layer.patch)
    return {"enc": layer.enc, "patch_off": layer.patch_off, "patch": state["patch"]}


def work(case):
    """Bytes: the compressed layer (mask, encrypted bits, patch offsets, scales; patch entries are a few per cent of
    these and left out), X and Y once each.  Operations: those of the product with the decoded matrix."""
    m, n, q, op = case["m"], case["n"], case["q"], case["op"]
    s = xe.get_sizes(m, n, case["n_in"], q, case["n_out"])
    packed = s["mask_words"] * 8 + s["enc_bytes"] + s["patch_off_words"] * 4 + q * m * 4
    if op in ("encode", "exhaustive"):
        return {"bytes": s["mask_words"] * 8 * (1 + q) + s["enc_bytes"] + s["patch_off_words"] * 4, "flops": 0}
    if op == "decode":
        out = {"planes": q * m * s["spr"] * 8, "f32": m * n * 4, "bf16": m * n * 2}[case["kind"]]
        return {"bytes": packed + out, "flops": 0}
    calls, B = case.get("calls", 1), case["B"]
    return {"bytes": calls * (packed + n * B * (4 if case["x"] == "f32" else 2) + m * B * 4), "flops": calls * 2 * m * n * B}


def tolerance(case):
    """Decoded values, encrypted bits and patches are defined bit for bit (Algorithm 1 and the search have one result; the
    planes of a dense value are added in a stated order).  Products are sums of fp32 terms whose order is free: 5e-8 to
    8e-8 from the 64-bit result.  With few columns of bf16 X the library may carry X as two 8-bit terms (1.5e-6 to
    2.3e-6, the truncation of the block-scaled instruction).  Both times four."""
    if case["op"] in ("spmm", "step"):
        return {"rel": 1e-5 if case["x"] == "bf16" and case["B"] <= 8 else 4e-7}
    return "exact"


# ------------------------------------------------------------------------------------- results in 64 bits

def _dense64(case, seed):
    keep, planes, alpha, _ = _weights(case, seed)
    w = torch.zeros(keep.shape, dtype=torch.float64, device=DEV)
    for p, b in enumerate(planes):
        w += torch.where(b, 1.0, -1.0).to(torch.float64) * alpha[p].to(torch.float64)[:, None]
    return torch.where(keep, w, torch.zeros((), dtype=torch.float64, device=DEV))


def exact(case, seed):
    op = case["op"]
    if op in ("encode", "exhaustive"):
        return None
    if op == "decode":
        if case["kind"] == "planes":
            m, spr = case["m"], -(-case["n"] // case["n_out"]) * (case["n_out"] // 64)
            _, planes, _, _ = _weights(case, _layer_seed(seed, 0))
            rows = [_words(b, case["n_out"]).view(-1, spr, 32).transpose(1, 2).reshape(-1, spr)[:m] for b in planes]
            return torch.stack([r.reshape(-1) for r in rows])
        return _dense64(case, _layer_seed(seed, 0))
    out = []
    for i in range(case.get("calls", 1)):
        s = _layer_seed(seed, i)
        out.append(_dense64(case, s) @ _x(case, s).to(torch.float64))
    return out if op == "step" else out[0]
