"""Workloads of the learned image codec that its speed is judged by.

A case is one pass through the library's public entry points on the GPU:

  op "layer"          one layer of the transforms, `Codec.run_layer`, on
                      device buffers (what a program that builds its own
                      pipeline, or replaces one stage of it, calls)
  op "encode_decode"  frames in device memory to bitstreams and back to
                      frames, `Codec.encode_decode`
  op "encode" / "decode"   one half of it

Models are the random-init weights of the repository's generator (N = 128
M = 192, and N = 192 M = 320); frames are its moving sinusoid fields with
noise; activations are drawn with the distribution that the normalisation
layers give for such weights.
"""
import functools
import math

import numpy as np
import torch

import synth
from paper_2208_01641_amd import Codec

PRECISION = {"fp32": 0, "bf16": 1, "e4m3": 2}
KIND = {"factorized": 0, "hyperprior": 1}

#: layer: (input grid, output grid) as divisors of the padded frame, kernel
#: size, stride, transposed, what follows.  Input channels "N" / "M" / 3.
LAYERS = {
    "GA0": (1, 2, 5, 2, False, "gdn", "3", "N"), "GA1": (2, 4, 5, 2, False, "gdn", "N", "N"),
    "GA2": (4, 8, 5, 2, False, "gdn", "N", "N"), "GA3": (8, 16, 5, 2, False, "quant", "N", "M"),
    "HA0": (16, 16, 3, 1, False, "relu", "M", "N"), "HA1": (16, 32, 5, 2, False, "relu", "N", "N"),
    "HA2": (32, 64, 5, 2, False, "quant", "N", "N"),
    "HS0": (64, 32, 5, 2, True, "relu", "N", "N"), "HS1": (32, 16, 5, 2, True, "relu", "N", "N"),
    "HS2": (16, 16, 3, 1, False, "index", "N", "M"),
    "GS0": (16, 8, 5, 2, True, "igdn", "M", "N"), "GS1": (8, 4, 5, 2, True, "igdn", "N", "N"),
    "GS2": (4, 2, 5, 2, True, "igdn", "N", "N"), "GS3": (2, 1, 5, 2, True, "image", "N", "3"),
}
TRANSFORM = ("GA0", "GA1", "GA2", "GA3", "GS0", "GS1", "GS2", "GS3")      # these run in the codec's precision
E4M3_OUT = ("GA0", "GA1", "GA2", "GS0", "GS1")                            # e4m3 form: activations stored as e4m3(8 v)
ACT_Q = 8.0                                                               # that scale, until a codec is calibrated


def listed():
    def layer(name, which, form, H, W, n=1, N=128, M=192):
        return {"name": name, "op": "layer", "layer": which, "form": form, "H": H, "W": W, "n": n, "N": N, "M": M}

    def call(name, op, model, form, H, W, n, N=128, M=192):
        return {"name": name, "op": op, "model": model, "form": form, "H": H, "W": W, "n": n, "N": N, "M": M}

    return [
        # one small image through the whole factorized-prior codec: latency of
        # a call, launches and hand-overs
        call("codec_128x128_factorized", "encode_decode", "factorized", "fp32", 128, 128, 1),
        # the ordinary use: a few 720p frames through the hyperprior codec
        call("codec_720p_hyperprior", "encode_decode", "hyperprior", "fp32", 720, 1280, 4),
        # the encoder takes in a 720p frame (bf16 form)
        layer("ga0_720p_bf16", "GA0", "bf16", 720, 1280),
        # the encoder's largest layer, 720p
        layer("ga1_720p_fp32", "GA1", "fp32", 720, 1280),
        # one 360p stream of a server: a grid that does not fill the chip
        layer("ga2_360p_fp32", "GA2", "fp32", 360, 640),
        # latents and symbols of a frame whose sides are no multiples of 64
        layer("ga3_470x834_fp32", "GA3", "fp32", 470, 834),
        # scale indices of a 720p frame (encoder and decoder both run it)
        layer("hs2_720p", "HS2", "fp32", 720, 1280),
        # synthesis of a 768 x 512 photograph in the e4m3 form
        layer("gs1_512x768_e4m3", "GS1", "e4m3", 512, 768),
        # the decoder's largest layer, 720p, in full and reduced precision
        layer("gs2_720p_fp32", "GS2", "fp32", 720, 1280),
        layer("gs2_720p_bf16", "GS2", "bf16", 720, 1280),
        # the same layer for a batch of four 1080p frames of the wide model
        layer("gs2_1080p_wide_e4m3", "GS2", "e4m3", 1080, 1920, 4, 192, 320),
        # reconstruction of a 720p frame
        layer("gs3_720p_fp32", "GS3", "fp32", 720, 1280),
    ]


def _cost(c):
    """Rough seconds of a case's matrix work on the unit its form runs on."""
    rate = {"fp32": 150e12, "bf16": 600e12, "e4m3": 1000e12}[c["form"]]
    if c.get("layer", "")[:2] in ("HA", "HS"):
        rate = 60e12
    return work(c)["flops"] / rate


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = max(_cost(c) for c in listed())
    form = rng.choice(["fp32", "fp32", "bf16", "e4m3"])
    H, W, n = log(64, 1088), log(64, 1920), rng.choice([1, 1, 1, 2, 3, 4])
    N, M = rng.choice([(128, 192), (128, 192), (192, 320)])
    if rng.random() < 0.75:
        c = {"op": "layer", "layer": rng.choice(sorted(LAYERS)), "form": form, "H": H, "W": W, "n": n, "N": N, "M": M}
    else:
        c = {"op": rng.choice(["encode", "decode", "encode_decode"]), "model": rng.choice(sorted(KIND)), "form": form,
             "H": min(H, 720), "W": min(W, 1280), "n": n, "N": 128, "M": 192}
    while _cost(c) > most:
        if c["n"] > 1:
            c["n"] -= 1
        else:
            c["H"], c["W"] = max(64, c["H"] * 3 // 4), max(64, c["W"] * 3 // 4)
    return c


# ------------------------------------------------------------------ the work
def _padded(c):
    return 64 * -(-c["H"] // 64), 64 * -(-c["W"] // 64)


def _grid(c, layer):
    """(input rows, columns, channels), (output rows, columns, channels)."""
    Hp, Wp = _padded(c)
    di, do, _, _, _, _, ci, co = LAYERS[layer]
    ch = {"N": c["N"], "M": c["M"], "3": 3}
    hi, wi = (c["H"], c["W"]) if di == 1 and ci == "3" else (Hp // di, Wp // di)
    ho, wo = (c["H"], c["W"]) if do == 1 and co == "3" else (Hp // do, Wp // do)
    return (hi, wi, ch[ci]), (ho, wo, ch[co])


def _layer_work(c, layer):
    Hp, Wp = _padded(c)
    di, do, k, _, transposed, post, _, _ = LAYERS[layer]
    (hi, wi, ci), (ho, wo, co) = _grid(c, layer)
    px = (Hp // di) * (Wp // di) if transposed else (Hp // do) * (Wp // do)
    mac = px * ci * co * k * k
    if post in ("gdn", "igdn"):
        mac += (Hp // do) * (Wp // do) * co * co
    act = {"fp32": 4, "bf16": 2, "e4m3": 1}[c["form"]] if layer in TRANSFORM else 4
    act_in, act_out = act, act
    if layer in ("GA0", "GA3") or layer[0] == "H":
        act_in = 4 if layer in ("GA0",) or layer[0] == "H" else act
        act_out = act if layer == "GA0" else 4
    if layer in ("GS0", "HS0"):
        act_in = 1
    if layer in ("HS2", "HA2"):
        act_out = 1
    if layer == "GA3":
        act_out = 5
    if c["form"] == "e4m3" and layer in ("GS2", "GS3"):
        act_in, act_out = (1, 2) if layer == "GS2" else (2, 4)
    if layer == "GS3":
        act_out = 4
    weights = ci * co * k * k * (act if layer in TRANSFORM else 4)
    return c["n"] * (hi * wi * ci * act_in + ho * wo * co * act_out) + weights, 2.0 * c["n"] * mac


def work(case):
    if case["op"] == "layer":
        b, f = _layer_work(case, case["layer"])
        return {"bytes": b, "flops": f}
    hyper = case["model"] == "hyperprior"
    enc = ["GA0", "GA1", "GA2", "GA3"] + (["HA0", "HA1", "HA2", "HS0", "HS1", "HS2"] if hyper else [])
    dec = (["HS0", "HS1", "HS2"] if hyper else []) + ["GS0", "GS1", "GS2", "GS3"]
    layers = (enc if case["op"] != "decode" else []) + (dec if case["op"] != "encode" else [])
    # frames in or out and the weights; what lies between stays on the chip
    frames = case["n"] * 12 * case["H"] * case["W"] * (2 if case["op"] == "encode_decode" else 1)
    weights = sum(4 * LAYERS[x][2] ** 2 * _grid(case, x)[0][2] * _grid(case, x)[1][2] for x in sorted(set(layers)))
    return {"bytes": frames + weights, "flops": sum(_layer_work(case, x)[1] for x in layers)}


# ---------------------------------------------------------------- the inputs
@functools.lru_cache(maxsize=4)
def _params(kind, N, M):
    return synth.model_params(kind, N, M, gamma="dense")


@functools.lru_cache(maxsize=4)
def _codec(kind, N, M, form, H, W, n, in_flight):
    # (a program keeps one handle per model and precision)
    return Codec(synth.weight_blob(_params(kind, N, M), kind, N, M), kind=kind, N=N, M=M, precision=PRECISION[form],
                 max_h=H, max_w=W, max_batch=n, max_in_flight=in_flight, entropy_threads=16, rans_lanes=8)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _frames(c, seed):
    return synth.frames_sinusoid_torch(c["H"], c["W"], range(c["n"]), stream=seed % (1 << 20))


def _activations(c, layer, seed):
    """A layer's input, in the layout and type it takes (NHWC)."""
    (hi, wi, ci), _ = _grid(c, layer)
    shape, g = (c["n"], hi, wi, ci), _generator(seed)
    if layer in ("GS0", "HS0"):                   # symbols: int8, a spread per channel
        spread = torch.empty((ci,), device="cuda").exponential_(0.5, generator=g)
        return torch.randn(shape, device="cuda", generator=g).mul_(spread).round_().clamp_(-64, 64).to(torch.int8)
    x = torch.randn(shape, device="cuda", generator=g)
    if layer in ("GA1", "GA2", "GA3"):            # after GDN
        x = x.mul_(2.0)
        x = x / (1.0 + 0.15 * x * x).sqrt()
    elif layer in ("GS1", "GS2", "GS3"):          # after IGDN
        x = x * (1.0 + 0.15 * x * x).sqrt()
    elif layer in ("HA1", "HA2", "HS1", "HS2"):   # after ReLU
        x = x.clamp_(min=0.0)
    if layer in TRANSFORM and c["form"] != "fp32":
        if c["form"] == "bf16" or layer == "GS3":
            return x.to(torch.bfloat16)
        return (ACT_Q * x).clamp_(-448, 448).to(torch.float8_e4m3fn)
    return x


def prepare(case, seed):
    c = case
    if c["op"] != "layer":
        kind = KIND[c["model"]]
        codec = _codec(kind, c["N"], c["M"], c["form"], c["H"], c["W"], 1, 6)
        x = _frames(c, seed)
        st = {"case": c, "codec": codec, "x": x, "out": torch.empty_like(x)}
        if c["op"] == "decode":
            st["streams"] = codec.encode(x)
        else:                                     # where the program sends its streams from
            st["bits"] = np.zeros((c["n"], codec.max_stream_bytes(c["H"], c["W"])), np.uint8)
            st["lens"] = np.zeros(c["n"], np.int64)
        return st
    layer = c["layer"]
    codec = _codec(1, c["N"], c["M"], c["form"], c["H"], c["W"], c["n"], 1)
    _, (ho, wo, co) = _grid(c, layer)
    x = _frames(c, seed) if layer == "GA0" else _activations(c, layer, seed)
    shape, aux, kind = (c["n"], ho, wo, co), None, torch.float32
    if layer == "GS3":
        shape = (c["n"], 3, ho, wo)
    elif layer in TRANSFORM and layer != "GA3":
        kind = {"fp32": torch.float32, "bf16": torch.bfloat16,
                "e4m3": torch.float8_e4m3fn if layer in E4M3_OUT else torch.bfloat16}[c["form"]]
    elif layer == "HS2":
        kind = torch.uint8
    if layer in ("GA3", "HA2"):                   # symbols; z itself is not needed, y is (h_a's input)
        aux = torch.empty(shape, dtype=torch.int8, device="cuda")
    out = None if layer == "HA2" else torch.empty(shape, dtype=kind, device="cuda")
    return {"case": c, "codec": codec, "x": x, "out": out, "aux": aux}


def run(state):
    c, codec = state["case"], state["codec"]
    if c["op"] == "layer":
        codec.run_layer(c["layer"], c["n"], c["H"], c["W"], state["x"], state["out"], state["aux"])
        return {k: state[k] for k in ("out", "aux") if state[k] is not None}
    if c["op"] == "decode":
        codec.decode(state["streams"], state["out"])
        return {"frames": state["out"]}
    bits = codec.encode(state["x"]) if c["op"] == "encode" else codec.encode_decode(state["x"], state["out"])
    for i, b in enumerate(bits):
        state["bits"][i, :len(b)] = np.frombuffer(b, np.uint8)
        state["lens"][i] = len(b)
    got = {"streams": state["bits"], "lengths": state["lens"]}
    if c["op"] == "encode_decode":
        got["frames"] = state["out"]
    return got


# ------------------------------------------------------- the same in 64 bits
def _conv64(x, w, b, stride):
    """x [n, H, W, ci], w [co, ci, k, k]: a strided convolution as one product per tap."""
    k = w.shape[2]
    n, H, W, ci = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2))
    ho, wo = -(-H // stride), -(-W // stride)
    y = b.expand(n * ho * wo, -1).clone()
    for u in range(k):
        for v in range(k):
            t = xp[:, u:u + stride * (ho - 1) + 1:stride, v:v + stride * (wo - 1) + 1:stride]
            y += t.reshape(-1, ci) @ w[:, :, u, v].t().contiguous()
    return y.view(n, ho, wo, -1)


def _deconv64(x, w, b):
    """x [n, H, W, ci], w [ci, co, 5, 5]: transposed convolution, stride 2, padding 2, output padding 1."""
    n, H, W, ci = x.shape
    co = w.shape[1]
    y = torch.zeros((n, 2 * H + 4, 2 * W + 4, co), dtype=x.dtype, device=x.device)
    flat = x.reshape(-1, ci)
    for u in range(5):
        for v in range(5):
            y[:, u:u + 2 * H:2, v:v + 2 * W:2] += (flat @ w[:, :, u, v].contiguous()).view(n, H, W, co)
    return y[:, 2:2 + 2 * H, 2:2 + 2 * W] + b


def exact(case, seed):
    if case["op"] != "layer":
        return None                               # integer decisions in the middle: no one value
    c, layer = case, case["layer"]
    _, _, _, stride, transposed, post, _, _ = LAYERS[layer]
    if post == "index" or layer == "HA2":
        return None                               # whole numbers only
    P = _params(1, c["N"], c["M"])
    w, b = (torch.from_numpy(P["%s.%s" % (layer.lower(), k)]).cuda().double() for k in "wb")
    Hp, Wp = _padded(c)
    if layer == "GA0":
        x = _frames(c, seed).double()
        x = torch.nn.functional.pad(x, (0, Wp - c["W"], 0, Hp - c["H"])).permute(0, 2, 3, 1).contiguous()
    else:
        x = _activations(c, layer, seed)
        scaled = x.dtype == torch.float8_e4m3fn
        x = x.double()
        if scaled:
            x = x / ACT_Q
        if layer == "HA0":
            x = x.abs()
        if layer == "HS0":
            x = x + torch.from_numpy(_medians(c)).cuda()
    y = _deconv64(x, w, b) if transposed else _conv64(x, w, b, stride)
    if post in ("gdn", "igdn"):
        beta, gamma = (torch.from_numpy(P["%s.%s" % (layer.lower(), k)]).cuda().double() for k in ("beta", "gamma"))
        co = y.shape[3]
        root = (beta + (y * y).view(-1, co) @ gamma.t().contiguous()).sqrt_().view(y.shape)
        y = y / root if post == "gdn" else y * root
        if c["form"] == "e4m3" and layer in E4M3_OUT:
            y = (ACT_Q * y).clamp(-448, 448)
    elif post == "relu":
        y = y.clamp(min=0.0)
    elif post == "image":
        y = y[:, :c["H"], :c["W"]].permute(0, 3, 1, 2).clamp(0.0, 1.0).contiguous()
    return {"out": y, "aux": None} if layer == "GA3" else {"out": y}


def _medians(c):
    """Medians of z's factorized densities (1-3-3-3-1 networks per channel), by bisection."""
    h = _params(1, c["N"], c["M"])["eb.density"]
    soft = lambda v: np.log1p(np.exp(v))          # noqa: E731
    lo, hi = np.full(len(h), -64.0), np.full(len(h), 64.0)

    def logit(x):
        u, at = x[:, None], 0
        for k, (din, dout) in enumerate(((1, 3), (3, 3), (3, 3), (3, 1))):
            m = soft(h[:, at:at + din * dout]).reshape(-1, dout, din)
            at += din * dout
            u = (m @ u[:, :, None])[:, :, 0] + h[:, at:at + dout]
            at += dout
            if k < 3:
                u = u + np.tanh(h[:, at:at + dout]) * np.tanh(u)
                at += dout
        return u[:, 0]

    for _ in range(80):
        mid = 0.5 * (lo + hi)
        up = logit(mid) < 0.0
        lo, hi = np.where(up, mid, lo), np.where(up, hi, mid)
    return (0.5 * (lo + hi)).astype(np.float32).astype(np.float64)
