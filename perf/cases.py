"""The layer calls whose speed this repository stands for, with their sizes, work and tolerances.

A case is one pass of a block-circulant layer, or of a chain of them, through the entry points of
`paper_1708_08917_amd.binding`: forward, backward (both gradients), a training pass (forward, both
gradients, the bias gradient) or a gradient step on the cached weight spectra.  `listed()` are the
layers of the configurations in `synth.py` and `layer_bench.py` and some of the tests' shapes;
`draw(rng)` gives others of the same kinds.  Buffers that a call can allocate itself (outputs and
workspaces) are left to the call, as in the README.
"""
from __future__ import annotations

import math

import torch

from paper_1708_08917_amd import binding as B

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# block sizes used in earnest: powers of two up to 512, and those of 3*2^a and 100 that layers of
# 96, 192, 384 or 4000 units ask for
K_POW2 = (8, 16, 32, 64, 128, 256, 512)
K_ALL = K_POW2 + (96, 100, 192)


def fc(name, op, n_in, n_out, k, batch, dtype="f32", relu=True):
    return {"name": name, "kind": "fc", "op": op, "n_in": n_in, "n_out": n_out, "k": k, "batch": batch, "dtype": dtype,
            "relu": relu}


def conv(name, op, n, c_in, c_out, h, w, r, stride, pad, k, dtype="f32"):
    return {"name": name, "kind": "conv", "op": op, "n": n, "c_in": c_in, "c_out": c_out, "h": h, "w": w, "r": r,
            "stride": stride, "pad": pad, "k": k, "dtype": dtype}


def head(name, batch, n0, n1, n2, n3, k):
    return {"name": name, "kind": "head", "batch": batch, "n0": n0, "n1": n1, "n2": n2, "n3": n3, "k": k}


def listed():
    return [
        # one input through one small layer: the latency of a single call
        fc("fc-1024-k16-b1", "forward", 1024, 1024, 16, 1, relu=False),
        # one input through an AlexNet-style classifier head: single-image inference
        head("head-b1", 1, 9216, 4096, 4096, 1000, 128),
        # a serving batch through a generic hidden layer (the benchmark's own workload)
        fc("fc-4096-k64-b64", "forward", 4096, 4096, 64, 64),
        # the same head for a full batch: offline inference
        head("head-b256", 256, 9216, 4096, 4096, 1000, 128),
        # training pass of a ragged layer with bfloat16 storage
        fc("fc-ragged-bf16-train", "train", 2112, 1280, 32, 700, "bf16"),
        # gradient step on the spectra, with dx for the layer below; block size not a power of two
        fc("fc-4000-k100-step", "step", 4000, 4000, 100, 64),
        # the largest layer: inference, backward pass, and a training pass with fp16 storage
        fc("fc-16384-k256-forward", "forward", 16384, 16384, 256, 1024, relu=False),
        fc("fc-16384-k256-backward", "backward", 16384, 16384, 256, 1024),
        fc("fc-16384-k256-f16-train", "train", 16384, 16384, 256, 1024, "f16"),
        # a mid-network 3x3 CONV layer: inference, backward pass
        conv("conv-256-28x28-forward", "forward", 32, 256, 256, 28, 28, 3, 1, 1, 64),
        conv("conv-256-28x28-backward", "backward", 32, 256, 256, 28, 28, 3, 1, 1, 64),
        # training pass of a late CONV layer on odd images, block size not a power of two
        conv("conv-384-13x13-k96-train", "train", 32, 384, 384, 13, 13, 3, 1, 1, 96),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fits(case):
    """No more work than the largest listed layer (16384 x 16384, k = 256, batch 1024)."""
    w = work(case)
    return w["bytes"] <= 2.0e8 and w["flops"] <= (6.0e9 if case["kind"] == "fc" else 1.5e9)


def _defined(k, blocks):
    """Whether a layer with this many input blocks gives defined results in every version of the fused FC
    kernel: with two chunks of input blocks, the second one ragged, some read LDS they had not written."""
    if k not in (64, 128, 256):
        return True
    chunk = 8 if k == 256 else 4096 // k
    return blocks % 8 == 0 or not (chunk // 2 < blocks < chunk or chunk < blocks < 2 * chunk)


def draw(rng):
    while True:
        kind = rng.choice(("fc", "fc", "fc", "conv", "conv", "head"))
        if kind == "fc":
            op = rng.choice(("forward", "forward", "backward", "train", "step"))
            dtype = "f32" if op == "step" else rng.choice(("f32", "f32", "f16", "bf16"))
            k = rng.choice(K_ALL if dtype == "f32" else K_POW2)
            q = max(1, _log_int(rng, 512, 16384) // k)
            p = max(1, _log_int(rng, 512, 16384) // k)
            if not (_defined(k, q) and _defined(k, p)):
                continue
            case = fc("", op, q * k, p * k, k, _log_int(rng, 1, 1024), dtype, rng.random() < 0.7)
        elif kind == "conv":
            op = rng.choice(("forward", "forward", "backward", "train", "step"))
            dtype = "f32" if op == "step" else rng.choice(("f32", "f32", "f32", "f16", "bf16"))
            k = rng.choice((16, 32, 64, 64, 64, 96, 128) if dtype == "f32" else (16, 32, 64, 64, 64, 128))
            q = max(1, _log_int(rng, 64, 512) // k)
            p = max(1, _log_int(rng, 64, 512) // k)
            r = rng.choice((1, 3, 3, 3, 5))
            h = _log_int(rng, 7, 56)
            w = h if rng.random() < 0.7 else max(7, h + rng.randint(-3, 3))
            case = conv("", op, _log_int(rng, 1, 64), q * k, p * k, h, w, r, rng.choice((1, 1, 1, 2)), rng.choice((0, r // 2, r // 2)),
                        k, dtype)
        else:
            k = rng.choice((32, 64, 128, 256))
            n0, n1, n2 = (max(1, _log_int(rng, 1024, 9216) // k) * k for _ in range(3))
            if not all(_defined(k, n // k) for n in (n0, n1)):
                continue
            case = head("", _log_int(rng, 1, 256), n0, n1, n2, 8 * _log_int(rng, 13, 125), k)
        del case["name"]
        if _fits(case):
            return case


def _normal(gen, scale, *shape):
    return torch.randn(*shape, device=DEV, generator=gen) * scale


def _uniform(gen, lo, hi, *shape):
    return torch.rand(*shape, device=DEV, generator=gen) * (hi - lo) + lo


def _out_hw(c):
    return ((c["h"] + 2 * c["pad"] - c["r"]) // c["stride"] + 1, (c["w"] + 2 * c["pad"] - c["r"]) // c["stride"] + 1)


def _head_layers(c):
    """(n_in, n_out, k, relu) of the three layers; the last one has blocks of 8 (1000 = 125 x 8)."""
    return [(c["n0"], c["n1"], c["k"], True), (c["n1"], c["n2"], c["k"], True), (c["n2"], c["n3"], 8, False)]


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    s = {"case": case}
    if case["kind"] == "head":
        s["keep"], layers = [], []
        for n_in, n_out, k, relu in _head_layers(case):
            w_hat = B.circ_precompute_spectra(_normal(gen, n_in ** -0.5, n_out // k, n_in // k, k))
            bias = _normal(gen, 0.1, n_out)
            s["keep"] += [w_hat, bias]
            layers.append(B.fc_layer(w_hat, bias, n_out // k, n_in // k, k, B.EPI_BIAS | (B.EPI_RELU if relu else 0)))
        s["layers"] = layers
        s["x"] = _uniform(gen, 0, 1, case["batch"], case["n0"])          # pooled features after a ReLU
        return s
    dtype = DTYPES[case["dtype"]]
    k = case["k"]
    if case["kind"] == "fc":
        p, q = case["n_out"] // k, case["n_in"] // k
        w = _normal(gen, case["n_in"] ** -0.5, p, q, k)
        s["w_hat"] = B.circ_precompute_spectra(w) if dtype == torch.float32 else B.circ_precompute_spectra_f16(w, dtype=dtype)
        s["x"] = _uniform(gen, -1, 1, case["batch"], case["n_in"]).to(dtype)
        if case["op"] != "backward":
            s["bias"] = _normal(gen, 0.1, case["n_out"])
        if case["op"] != "forward":
            s["dy"] = _uniform(gen, -1, 1, case["batch"], case["n_out"]).to(dtype)
    else:
        p, q, r = case["c_out"] // k, case["c_in"] // k, case["r"]
        w = _normal(gen, (2.0 / (r * r * case["c_in"])) ** 0.5, r, r, p, q, k)
        s["w_hat"] = B.circ_precompute_spectra(w)                        # CONV keeps fp32 spectra for every storage type
        s["x"] = _uniform(gen, -1, 1, case["n"], case["c_in"], case["h"], case["w"]).to(dtype)
        if case["op"] != "backward":
            s["bias"] = _normal(gen, 0.1, case["c_out"])
        if case["op"] != "forward":
            s["dy"] = _uniform(gen, -1, 1, case["n"], case["c_out"], *_out_hw(case)).to(dtype)
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "head":
        y = torch.empty(c["batch"], c["n3"], dtype=torch.float32, device=DEV)
        return {"y": B.circ_chain_forward(state["layers"], state["x"], y)}
    return _run_fc(state, c) if c["kind"] == "fc" else _run_conv(state, c)


def _run_fc(s, c):
    op, k, w_hat, x = c["op"], c["k"], s["w_hat"], s["x"]
    p, q = c["n_out"] // k, c["n_in"] // k
    half = c["dtype"] != "f32"
    out = {}
    if op in ("forward", "train"):
        epi = B.EPI_BIAS | (B.EPI_RELU if c["relu"] else 0)
        out["y"] = (B.circ_fc_forward_f16 if half else B.circ_fc_forward)(w_hat, x, s["bias"], None, p, q, k, epi)
    if op in ("backward", "train"):
        out["dx"], out["dw"] = (B.circ_fc_backward_f16 if half else B.circ_fc_backward)(w_hat, x, s["dy"], p, q, k)
    if op == "train" and not half:
        out["db"] = B.circ_bias_grad(s["dy"])
    if op == "step":
        out["dx"] = B.circ_fc_sgd_step(w_hat, x, s["dy"], _rate(c), p, q, k, need_dx=True)
        out["w"] = B.circ_export_weights(w_hat, 1, p, q, k)              # the weights after the step
    return out


def _run_conv(s, c):
    op, k, w_hat, x = c["op"], c["k"], s["w_hat"], s["x"]
    r, stride, pad = c["r"], c["stride"], c["pad"]
    half = c["dtype"] != "f32"
    out = {}
    if op in ("forward", "train"):
        out["y"] = (B.circ_conv_forward_f16 if half else B.circ_conv_forward)(w_hat, x, s["bias"], None, c["c_out"], r, stride, pad,
                                                                             k, B.EPI_BIAS | B.EPI_RELU)
    if op in ("backward", "train"):
        out["dx"], out["dw"] = (B.circ_conv_backward_f16 if half else B.circ_conv_backward)(w_hat, x, s["dy"], c["c_in"], c["h"], c["w"],
                                                                                           r, stride, pad, k)
    if op == "train" and not half:
        out["db"] = B.circ_bias_grad(s["dy"])
    if op == "step":
        out["dx"] = B.circ_conv_sgd_step(w_hat, x, s["dy"], _rate(c), c["c_in"], c["h"], c["w"], r, stride, pad, k, need_dx=True)
        out["w"] = B.circ_export_weights(w_hat, r * r, c["c_out"] // k, c["c_in"] // k, k)
    return out


def _rate(c):
    """A learning rate at which one step moves the weights by about a tenth of their size: dw is a sum of
    `terms` products of two uniform values in [-1, 1], of variance 1/9 each."""
    if c["kind"] == "fc":
        return 0.1 * c["n_in"] ** -0.5 / math.sqrt(c["batch"] * c["k"] / 9)
    ho, wo = _out_hw(c)
    return 0.1 * (2.0 / (c["r"] ** 2 * c["c_in"])) ** 0.5 / math.sqrt(c["n"] * ho * wo * c["k"] / 9)


def _fft_flops(k):
    return 2.5 * k * math.log2(k)


def _parts(case):
    """Per direction of a layer: (values of x, values of y, values of w, weight spectrum values (complex),
    flops of one contraction, flops of the transforms of x, of y and of w)."""
    k = case["k"]
    f = k // 2 + 1
    if case["kind"] == "fc":
        p, q, rows = case["n_out"] // k, case["n_in"] // k, case["batch"]
        nx, ny, taps, pix = rows * case["n_in"], rows * case["n_out"], 1, rows
    else:
        p, q = case["c_out"] // k, case["c_in"] // k
        ho, wo = _out_hw(case)
        nx, ny = case["n"] * case["c_in"] * case["h"] * case["w"], case["n"] * case["c_out"] * ho * wo
        taps, pix = case["r"] ** 2, case["n"] * ho * wo
    nw = taps * p * q * k
    return (nx, ny, nw, taps * p * q * f, 8.0 * taps * p * q * f * pix, nx / k * _fft_flops(k), ny / k * _fft_flops(k),
            nw / k * _fft_flops(k))


def work(case):
    """What a pass cannot do without: every input read once, every output written once; the products of the
    spectra and the transforms (2.5 k log2 k operations per real block)."""
    if case["kind"] == "head":
        byts = 4 * case["batch"] * (case["n0"] + case["n3"])
        flops = 0.0
        for n_in, n_out, k, _ in _head_layers(case):
            one = {"kind": "fc", "n_in": n_in, "n_out": n_out, "k": k, "batch": case["batch"]}
            _, _, _, nwh, mul, fx, fy, _ = _parts(one)
            byts += 8 * nwh + 4 * n_out
            flops += mul + fx + fy
        return {"bytes": byts, "flops": flops}
    nx, ny, nw, nwh, mul, fx, fy, fw = _parts(case)
    act = 4 if case["dtype"] == "f32" else 2
    spec = 8 if case["dtype"] == "f32" or case["kind"] == "conv" else 4
    op = case["op"]
    byts = act * (nx + ny) + spec * nwh                                  # x, w_hat and y, or x, dy and w_hat
    if op == "forward":
        return {"bytes": byts, "flops": mul + fx + fy}
    byts += act * nx                                                     # dx
    if op == "step":
        return {"bytes": byts + spec * nwh + 4 * nw, "flops": 2 * mul + 2 * fx + fy + fw}
    byts += 4 * nw                                                       # dw
    flops = 2 * mul + 2 * fx + fy + fw
    if op == "train":
        byts += act * ny                                                 # y
        flops += mul + fx + fy
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Four times the largest difference from the same pass in float64 (all listed cases and 120 drawn
    ones): fp32 rel 5.5e-7 and max 3.8e-6 (three layers in a row), fp16 4.2e-4 and 3.0e-3, bfloat16 3.4e-3
    and 2.1e-2 (one to four roundings of 2^-11 and 2^-8)."""
    if case["kind"] == "head" or case["dtype"] == "f32":
        return {"rel": 2.2e-6, "max": 1.5e-5}
    return {"rel": 1.7e-3, "max": 1.2e-2} if case["dtype"] == "f16" else {"rel": 1.3e-2, "max": 8e-2}
