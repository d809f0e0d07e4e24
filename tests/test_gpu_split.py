"""Small grids: the split-K kernels at each of their tile shapes, whole tensors
against the same layer in float64.

Sizes give grids from less than one tile to those where 32-pixel tiles begin,
with pixel groups that run past the last pixel or across images.  The
reference takes the operands as the form rounds them, so what is left is FP32
accumulation (1e-4 of max |ref|) and one rounding of a stored bf16 (2^-8) or
e4m3 (2^-4) output; integer outputs must be the decision taken on the layer's
own float output.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dims
from test_gpu_fp8 import FP8_OUT_TOL, w_fp8
from test_gpu_precision import BF16_OUT_TOL, bf16
from test_gpu_staged import ACT_Q, conv64, deconv64

pytestmark = pytest.mark.gpu

FP32, BF16, FP8 = 0, 1, 2
# (precision, layer, N, M, n, H, W)
CASES = [
    # GDN layers: 16- and 32-pixel tiles, 128 and 192 rows
    (FP32, "GA1", 128, 192, 1, 64, 64), (FP32, "GA2", 128, 192, 1, 64, 128), (FP32, "GA2", 128, 192, 3, 64, 64),
    (FP32, "GA1", 128, 192, 5, 256, 320), (FP32, "GS0", 128, 192, 3, 64, 64), (FP32, "GS1", 128, 192, 5, 128, 192),
    (FP32, "GS2", 128, 192, 1, 64, 128), (FP32, "GA1", 192, 320, 1, 64, 128), (FP32, "GS0", 192, 320, 3, 64, 192),
    (FP32, "GS1", 192, 320, 4, 256, 320),
    (BF16, "GA1", 128, 192, 1, 64, 64), (BF16, "GA2", 128, 192, 3, 64, 64), (BF16, "GA1", 128, 192, 5, 256, 320),
    (BF16, "GS0", 128, 192, 3, 64, 64), (BF16, "GS1", 192, 320, 1, 128, 192), (BF16, "GS0", 192, 320, 5, 256, 320),
    (FP8, "GA1", 128, 192, 1, 64, 64), (FP8, "GA2", 128, 192, 3, 64, 64), (FP8, "GS1", 128, 192, 1, 512, 768),
    (FP8, "GS2", 128, 192, 1, 64, 128), (FP8, "GA2", 192, 320, 3, 64, 192), (FP8, "GS1", 192, 320, 5, 256, 320),
    # g_a's last layer, symbols
    (FP32, "GA3", 128, 192, 3, 64, 64), (FP32, "GA3", 128, 192, 1, 448, 832), (FP32, "GA3", 128, 192, 1, 704, 1280),
    (FP32, "GA3", 192, 320, 6, 704, 1280), (BF16, "GA3", 128, 192, 3, 64, 64), (BF16, "GA3", 128, 192, 1, 704, 1280),
    (FP8, "GA3", 128, 192, 3, 64, 64), (FP8, "GA3", 128, 192, 1, 704, 1280), (FP8, "GA3", 192, 320, 1, 192, 320),
    # hyper layers
    (FP32, "HA0", 128, 192, 1, 64, 64), (FP32, "HA0", 128, 192, 5, 704, 1280), (FP32, "HA1", 128, 192, 3, 192, 320),
    (FP32, "HA1", 192, 320, 1, 704, 1280), (FP32, "HA2", 128, 192, 3, 64, 64), (FP32, "HS0", 128, 192, 3, 64, 64),
    (FP32, "HS0", 192, 320, 1, 704, 1280), (FP32, "HS1", 128, 192, 1, 704, 1280), (FP32, "HS2", 128, 192, 3, 64, 64),
    (FP32, "HS2", 128, 192, 1, 448, 832), (FP32, "HS2", 192, 320, 1, 1088, 1920),
]
SHAPE = {  # input and output divisor of the padded frame
    "GA1": (2, 4), "GA2": (4, 8), "GA3": (8, 16), "GS0": (16, 8), "GS1": (8, 4), "GS2": (4, 2), "HA0": (16, 16),
    "HA1": (16, 32), "HA2": (32, 64), "HS0": (64, 32), "HS1": (32, 16), "HS2": (16, 16)}


def conv3(torch, x, w, b):
    n, H, W, ci = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b.expand(n * H * W, -1).clone()
    for u in range(3):
        for v in range(3):
            y += xp[:, u:u + H, v:v + W].reshape(-1, ci) @ w[:, :, u, v].t().contiguous()
    return y.view(n, H, W, -1)


@pytest.mark.parametrize("prec,layer,N,M,n,H,W", CASES)
def test_split_layer(prec, layer, N, M, n, H, W):
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    di, do = SHAPE[layer]
    hi, wi, ho, wo = d["Hp"] // di, d["Wp"] // di, d["Hp"] // do, d["Wp"] // do
    name = layer.lower()
    up, gdn, hyper = layer[1] == "S" and layer != "HS2", layer in ("GA1", "GA2", "GS0", "GS1", "GS2"), layer[0] == "H"
    w = P[name + ".w"]
    ci, co = (w.shape[0], w.shape[1]) if up else (w.shape[1], w.shape[0])
    g = torch.Generator(device="cuda")
    g.manual_seed(hi * wi + n)
    x = torch.randn((n, hi, wi, ci), device="cuda", generator=g)
    kind = 1
    symbols = layer in ("GS0", "HS0")
    c = Codec(synth.weight_blob(P, kind, N, M), kind=kind, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)
    if symbols:
        x = (3 * x).round().clamp(-64, 64).to(torch.int8)
        ref_in = x.double()
        if layer == "HS0":
            ref_in = ref_in + torch.from_numpy(c.medians().astype(np.float64)).cuda()
    elif prec == FP8 and not hyper:
        x = (ACT_Q * x).to(torch.float8_e4m3fn)
        ref_in = x.double() / ACT_Q
    else:
        x = x.to(torch.bfloat16) if prec == BF16 and not hyper else x
        ref_in = x.double()
    if layer == "HA0":
        ref_in = ref_in.abs()
    if not hyper and prec != FP32:
        w = bf16(w) if prec == BF16 or symbols else w_fp8(w, "deconv" if up else "conv")
    w, b = (torch.from_numpy(np.asarray(t, np.float64)).cuda() for t in (w, P[name + ".b"]))
    assert c.layer_kernel(layer, H, W)[1] > 1
    ref = deconv64(torch, ref_in, w, b) if up else conv3(torch, ref_in, w, b) if w.shape[2] == 3 else conv64(torch, ref_in, w, b)
    if gdn:
        beta, gamma = (torch.from_numpy(np.asarray(P[name + k], np.float64)).cuda() for k in (".beta", ".gamma"))
        norm = (beta + (ref * ref).view(-1, co) @ gamma.t().contiguous()).sqrt().view(ref.shape)
        ref = ref * norm if up else ref / norm
    elif layer in ("HA0", "HA1", "HS0", "HS1"):
        ref = ref.clamp(min=0.0)
    out_dt = torch.float32
    if gdn and prec != FP32:
        out_dt = torch.bfloat16 if prec == BF16 or layer == "GS2" else torch.float8_e4m3fn
    val = torch.empty((n, ho, wo, co), dtype=out_dt, device="cuda")
    ints = torch.empty((n, ho, wo, co), dtype=torch.uint8 if layer == "HS2" else torch.int8, device="cuda")
    if layer == "HS2":
        c.run_layer(layer, n, H, W, x, ints, val)
    else:
        c.run_layer(layer, n, H, W, x, val, ints if layer in ("GA3", "HA2") else None)
    got = val.double() / (ACT_Q if out_dt == torch.float8_e4m3fn else 1.0)
    err = float((got - ref).abs().max() / ref.abs().max())
    tol = 1e-4 if out_dt == torch.float32 else BF16_OUT_TOL if out_dt == torch.bfloat16 else FP8_OUT_TOL
    assert err < tol, f"max error / max |ref| = {err:.2e}"
    v = val.cpu().numpy() if out_dt == torch.float32 else None
    if layer == "HS2":
        assert np.array_equal(ints.cpu().numpy(), oracle.scale_index_f32(v, 1).reshape(v.shape))
    elif layer in ("GA3", "HA2"):
        mu = c.medians() if layer == "HA2" else np.float32(0)
        assert np.array_equal(ints.cpu().numpy(), np.clip(np.rint(v - mu), -64, 64).astype(np.int8))
    c.close()


# (layer, N, M, images of the batch, H, W, norm): alone the layer takes two passes
# (sums in blocks of 16 or of 32 rows, then the normalisation), the batch one
TWO_PASS = [("GA1", 128, 192, 9, 64, 64, 0), ("GA2", 128, 192, 33, 64, 64, 1), ("GA2", 128, 192, 2, 256, 320, 0),
            ("GS0", 128, 192, 33, 64, 64, 0), ("GS1", 128, 192, 10, 64, 64, 1), ("GS1", 128, 192, 2, 128, 192, 0),
            ("GS2", 128, 192, 3, 64, 64, 0), ("GA1", 192, 320, 11, 64, 64, 0), ("GA2", 192, 320, 2, 320, 448, 1),
            ("GS0", 192, 320, 11, 64, 192, 1), ("GS1", 192, 320, 2, 192, 192, 0)]


# reduced forms, the same layout: alone on the split-K kernels, the batch on the staged
# ones with four K slots; grids whose last block is not full
FOUR_SUMS = [(BF16, "GA1", 128, 192, 41, 64, 64, 0), (BF16, "GA2", 128, 192, 54, 64, 192, 1), (BF16, "GS0", 128, 192, 161, 64, 64, 0),
             (BF16, "GS1", 128, 192, 41, 64, 64, 0), (BF16, "GS2", 128, 192, 3, 128, 192, 0), (BF16, "GA1", 192, 320, 14, 128, 192, 0),
             (BF16, "GS0", 192, 320, 27, 64, 384, 1), (BF16, "GS2", 192, 320, 11, 64, 64, 0), (FP8, "GA1", 128, 192, 25, 64, 64, 1),
             (FP8, "GA2", 128, 192, 33, 64, 192, 0), (FP8, "GS1", 128, 192, 25, 64, 64, 0), (FP8, "GS2", 128, 192, 3, 128, 192, 1),
             (FP8, "GA2", 192, 320, 33, 64, 192, 0), (FP8, "GS1", 192, 320, 9, 128, 192, 0)]


@pytest.mark.parametrize("prec,layer,N,M,n,H,W,norm", [(FP32,) + c for c in TWO_PASS] + FOUR_SUMS)
def test_batch_route_same_bits(prec, layer, N, M, n, H, W, norm):
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    di, do = SHAPE[layer]
    ci = M if layer == "GS0" else N
    g = torch.Generator(device="cuda")
    g.manual_seed(N + n)
    x = torch.randn((n, d["Hp"] // di, d["Wp"] // di, ci), device="cuda", generator=g)
    if layer == "GS0":
        x = (3 * x).round().clamp(-64, 64).to(torch.int8)
    elif prec != FP32:
        x = x.to(torch.bfloat16) if prec == BF16 else (ACT_Q * x).to(torch.float8_e4m3fn)
    out_dt = torch.float32 if prec == FP32 else torch.bfloat16 if prec == BF16 or layer == "GS2" else torch.float8_e4m3fn
    out = torch.empty((n, d["Hp"] // do, d["Wp"] // do, N), dtype=out_dt, device="cuda")
    one = torch.empty((1,) + out.shape[1:], dtype=out_dt, device="cuda")
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1, norm=norm)
    c.run_layer(layer, n, H, W, x, out)
    assert bool(out.float().isfinite().all())
    for i in range(n):
        c.run_layer(layer, 1, H, W, x[i:i + 1].contiguous(), one)
        assert torch.equal(out[i].view(torch.uint8), one[0].view(torch.uint8)), f"image {i} of {n} differs"
    c.close()
