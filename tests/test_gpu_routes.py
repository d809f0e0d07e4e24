"""Every kernel and tile that a layer can take (up to 5 million pixels): against
float64, against the same image alone, and with a NaN that must reach exactly
the outputs whose window holds it.

References take the operands as the form rounds them, so what is left is FP32
accumulation (1e-4 of max |ref|) and one rounding of a stored bf16 (2^-8) or e4m3
(2^-4) output.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dims
from route_util import CONTEXT, GDN, MODELS, routes, tile
from test_gpu_fp8 import FP8_OUT_TOL, w_fp8
from test_gpu_precision import BF16_OUT_TOL, bf16
from test_gpu_split import SHAPE, conv3
from test_gpu_staged import ACT_Q, conv64, deconv64

pytestmark = pytest.mark.gpu

FP32, BF16, FP8 = 0, 1, 2
ROUTES = [(kind, N, M, p, layer) for kind, N, M, p, layers in MODELS for layer in layers if layer not in ("GA0", "GS3")]


def grids(layer, H, W):
    d = dims(H, W)
    di, do = SHAPE.get(layer, (16, 16))
    return d["Hp"] // di, d["Wp"] // di, d["Hp"] // do, d["Wp"] // do


def codec(kind, N, M, prec, P=None):
    from paper_2208_01641_amd import Codec
    P = P or synth.model_params(kind, N, M, gamma="dense")
    return Codec(synth.weight_blob(P, kind, N, M), kind=kind, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)


def activations(torch, kind, prec, layer, shape, seed):
    """(the layer's input, what it stands for in float64)"""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(shape, device="cuda", generator=g)
    if layer == "HS0" or (layer == "GS0" and kind != 2):
        x = (3 * x).round().clamp(-64, 64).to(torch.int8)
    elif layer[0] in "HCE" or prec == FP32:
        pass
    elif prec == BF16 or layer == "GS0":
        x = x.to(torch.bfloat16)
    else:
        x = (ACT_Q * x).to(torch.float8_e4m3fn)
        return x, lambda t: t.double() / ACT_Q
    return x, lambda t: t.double()


def out_type(torch, prec, layer):
    if layer not in GDN or prec == FP32:
        return torch.uint8 if layer == "HS2" else torch.float32
    return torch.bfloat16 if prec == BF16 or layer == "GS2" else torch.float8_e4m3fn


def reference(torch, c, P, prec, layer, kind, N, x):
    name, up = layer.lower(), layer[1] == "S" and layer != "HS2"
    w = P[name + ".w"]
    if prec != FP32:
        w = bf16(w) if prec == BF16 or layer == "GS0" else w_fp8(w, "deconv" if up else "conv")
    w, b = (torch.from_numpy(np.asarray(t, np.float64)).cuda() for t in (w, P[name + ".b"]))
    if layer == "HA0" and kind == 1:
        x = x.abs()
    if layer == "HS0":
        x = x + torch.from_numpy(c.medians().astype(np.float64)).cuda()
    ref = deconv64(torch, x, w, b) if up else conv3(torch, x, w, b) if w.shape[2] == 3 else conv64(torch, x, w, b)
    if layer in GDN:
        beta, gamma = (torch.from_numpy(np.asarray(P[name + k], np.float64)).cuda() for k in (".beta", ".gamma"))
        norm = (beta + (ref * ref).view(-1, N) @ gamma.t().contiguous()).sqrt().view(ref.shape)
        ref = ref * norm if up else ref / norm
    elif layer in ("HA0", "HA1", "HS0", "HS1"):
        ref = ref.clamp(min=0.0)
    return ref


@pytest.mark.parametrize("kind,N,M,prec,layer", ROUTES)
def test_every_route(kind, N, M, prec, layer):
    import torch
    P = synth.model_params(kind, N, M, gamma="dense")
    c = codec(kind, N, M, prec, P)
    ci = {"HA0": M, "GS0": M, "CX": M, "EP0A": 4 * M, "EP1A": 640, "EP2A": 512}.get(layer, N)
    co = {"GA3": M, "HS2": M if kind == 1 else 2 * M, "CX": 2 * M, "EP0A": 640, "EP1A": 512, "EP2A": M}.get(layer, N)
    for t, (n, H, W) in routes(kind, N, M, prec, layer).items():
        if t[0] == "direct":
            continue
        hi, wi, ho, wo = grids(layer, H, W)
        what = f"{layer} {t} at {n} x {H} x {W}"
        x, value = activations(torch, kind, prec, layer, (n, hi, wi, ci), n * H + W)
        wide = layer == "CX" or (layer == "HS2" and kind == 2)            # half of [psi; ctx]
        shape = (ho, wo, 4 * M if wide else co)
        y2 = torch.randn((n, hi, wi, M), device="cuda") if layer == "EP2A" else None

        def run(x, y2):
            out = torch.zeros((len(x),) + shape, dtype=torch.uint8 if layer == "EP2A" else out_type(torch, prec, layer), device="cuda")
            if wide:
                out = out.float()
            aux = None
            if layer in ("GA3", "HA2", "EP2A"):
                aux = torch.zeros((len(x),) + shape, dtype=torch.int8, device="cuda")
            elif layer == "HS2" and kind == 1:
                aux = torch.zeros((len(x),) + shape, device="cuda")
            yq = torch.zeros_like(y2) if y2 is not None else None
            c.run_layer(layer, len(x), H, W, x, out, aux, y2, yq)
            return [v for v in (out, aux, yq) if v is not None]

        got = run(x, y2)
        last = run(x[n - 1:].contiguous(), y2[n - 1:].contiguous() if y2 is not None else None)
        for a, b in zip(got, last):
            assert torch.equal(a[n - 1].view(torch.uint8), b[0].view(torch.uint8)), what + ": not the bits of the image alone"
        if layer in CONTEXT or wide:
            continue
        ref = reference(torch, c, P, prec if layer[0] == "G" else FP32, layer, kind, N, value(x[n - 1:]))
        val = (last[1] if layer == "HS2" else last[0])
        e4m3 = val.dtype == torch.float8_e4m3fn
        if e4m3:
            ref = ref.clamp(-448 / ACT_Q, 448 / ACT_Q)
        err = float((val.double() / (ACT_Q if e4m3 else 1.0) - ref).abs().max() / ref.abs().max())
        assert err < (1e-4 if val.dtype == torch.float32 else FP8_OUT_TOL if e4m3 else BF16_OUT_TOL), f"{what}: {err:.2e}"
        if layer == "HS2":
            v = val.cpu().numpy()
            assert np.array_equal(last[0].cpu().numpy(), oracle.scale_index_f32(v, 1).reshape(v.shape)), what
        elif layer in ("GA3", "HA2"):
            mu = c.medians() if layer == "HA2" else np.float32(0)
            assert np.array_equal(last[1].cpu().numpy(), np.clip(np.rint(val.cpu().numpy() - mu), -64, 64).astype(np.int8)), what
    c.close()


@pytest.mark.parametrize("kind,N,M,prec,layer", [r for r in ROUTES if r[4] in GDN and r[3] != FP8 and (r[0] == 2 or r[4] != "GS0")])
def test_a_nan_reaches_its_window(kind, N, M, prec, layer):
    """The contraction over channels spreads a NaN over its pixel; a tap outside
    the image, a halo or a padded chunk that held it would spread it further."""
    import torch
    c = codec(kind, N, M, prec)
    ci = M if layer == "GS0" else N
    for t, (n, H, W) in routes(kind, N, M, prec, layer).items():
        if t[0] == "direct":
            continue
        hi, wi, ho, wo = grids(layer, H, W)
        x, _ = activations(torch, kind, prec, layer, (n, hi, wi, ci), n + H + W)
        out = torch.empty((n, ho, wo, N), dtype=out_type(torch, prec, layer), device="cuda")
        c.run_layer(layer, n, H, W, x, out)
        assert bool(out.isfinite().all())
        reached = torch.zeros((n, ho, wo), dtype=torch.bool, device="cuda")
        for i, y, xx, ch in ((0, 0, 0, 0), (n - 1, hi - 1, wi - 1, ci - 1), (n // 2, hi // 2, wi // 3, ci // 2), (0, hi - 1, 0, 31)):
            x[i, y, xx, ch] = float("nan")
            if layer[1] == "S":                                # output 2 y - 2 .. 2 y + 2
                reached[i, max(2 * y - 2, 0):2 * y + 3, max(2 * xx - 2, 0):2 * xx + 3] = True
            else:                                              # outputs whose window 2 o - 2 .. 2 o + 2 holds y
                reached[i, max(-(-(y - 2) // 2), 0):(y + 2) // 2 + 1, max(-(-(xx - 2) // 2), 0):(xx + 2) // 2 + 1] = True
        got = torch.empty_like(out)
        c.run_layer(layer, n, H, W, x, got)
        what = f"{layer} {t} at {n} x {H} x {W}"
        assert bool(got[reached].isnan().all()), what
        assert torch.equal(got[~reached].view(torch.uint8), out[~reached].view(torch.uint8)), what
    c.close()
