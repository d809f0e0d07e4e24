"""GDN layers on the kernels that stage both operands in LDS (whole frames and
batches): whole tensors against the same layer in float64.

Sizes are those where the staged kernels begin (half a wave per SIMD), where
one 16-pixel tile per wave gives way to two, and grids whose last block is
not full or whose blocks cross from one image to the next.  The reference
takes the operands as the form rounds them (bf16 or per-row-scaled e4m3
weights, the stored activations), so what is left is FP32 accumulation (1e-4
of max |ref|) and one rounding of the stored output (bf16 2^-8, e4m3 2^-4).
"""
import numpy as np
import pytest

import synth
from gpu_util import dims
from test_gpu_fp8 import FP8_OUT_TOL, w_fp8
from test_gpu_precision import BF16_OUT_TOL, bf16

pytestmark = pytest.mark.gpu

FP32, BF16, FP8 = 0, 1, 2
# (precision, layer, N, M, n, H, W)
CASES = [
    (FP32, "GA1", 128, 192, 3, 320, 448), (FP32, "GA2", 128, 192, 5, 832, 704), (FP32, "GS0", 128, 192, 1, 512, 1024),
    (FP32, "GS1", 128, 192, 1, 320, 448), (FP32, "GS2", 128, 192, 2, 320, 448), (FP32, "GS2", 192, 320, 1, 576, 960),
    (FP32, "GS0", 192, 320, 1, 1024, 1088),
    (BF16, "GA1", 128, 192, 3, 320, 448), (BF16, "GA2", 128, 192, 5, 832, 704), (BF16, "GS0", 128, 192, 1, 512, 1024),
    (BF16, "GS1", 128, 192, 1, 320, 448), (BF16, "GS2", 192, 320, 1, 576, 960), (BF16, "GS0", 192, 320, 1, 1024, 1088),
    (FP8, "GA1", 128, 192, 1, 704, 768), (FP8, "GA2", 128, 192, 5, 832, 704), (FP8, "GS0", 128, 192, 1, 512, 1024),
    (FP8, "GS1", 128, 192, 1, 704, 768), (FP8, "GS2", 192, 320, 1, 576, 960), (FP8, "GA1", 192, 320, 3, 512, 576),
]
ACT_Q = 8.0        # e4m3 activations hold 8 x the value until a codec is calibrated


def conv64(torch, x, w, b):
    """x [n, H, W, ci], w [co, ci, 5, 5]: stride 2, padding 2."""
    n, H, W, ci = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 2, 2, 2, 2))
    y = b.expand(n * (H // 2) * (W // 2), -1).clone()
    for u in range(5):
        for v in range(5):
            y += xp[:, u:u + H - 1:2, v:v + W - 1:2].reshape(-1, ci) @ w[:, :, u, v].t().contiguous()
    return y.view(n, H // 2, W // 2, -1)


def deconv64(torch, x, w, b):
    """x [n, H, W, ci], w [ci, co, 5, 5]: stride 2, padding 2, output padding 1."""
    n, H, W, ci = x.shape
    y = torch.zeros((n, 2 * H + 4, 2 * W + 4, w.shape[1]), dtype=x.dtype, device=x.device)
    for u in range(5):
        for v in range(5):
            y[:, u:u + 2 * H:2, v:v + 2 * W:2] += (x.reshape(-1, ci) @ w[:, :, u, v].contiguous()).view(n, H, W, -1)
    return y[:, 2:2 + 2 * H, 2:2 + 2 * W] + b


@pytest.mark.parametrize("prec,layer,N,M,n,H,W", CASES)
def test_staged_layer(prec, layer, N, M, n, H, W):
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    den = {"GA1": 2, "GA2": 4, "GS0": 16, "GS1": 8, "GS2": 4}[layer]
    up = layer[1] == "S"
    hi, wi, ci = d["Hp"] // den, d["Wp"] // den, M if layer == "GS0" else N
    ho, wo = (2 * hi, 2 * wi) if up else (hi // 2, wi // 2)
    g = torch.Generator(device="cuda")
    g.manual_seed(hi * wi + n)
    x = torch.randn((n, hi, wi, ci), device="cuda", generator=g)
    name = layer.lower()
    first = layer == "GS0"                                     # symbols, bf16 weights in the e4m3 form too
    if first:
        x = (3 * x).round().clamp(-64, 64).to(torch.int8)
        ref_in = x.double()
    elif prec == FP8:
        x = (ACT_Q * x).to(torch.float8_e4m3fn)
        ref_in = x.double() / ACT_Q
    else:
        x = x.to(torch.bfloat16) if prec == BF16 else x
        ref_in = x.double()
    w = P[name + ".w"]
    w = w if prec == FP32 else bf16(w) if prec == BF16 or first else w_fp8(w, "deconv" if up else "conv")
    w, b, beta, gamma = (torch.from_numpy(np.asarray(t, np.float64)).cuda()
                         for t in (w, P[name + ".b"], P[name + ".beta"], P[name + ".gamma"]))
    out_dt = torch.float32 if prec == FP32 else torch.bfloat16 if prec == BF16 or layer == "GS2" else torch.float8_e4m3fn
    out = torch.empty((n, ho, wo, N), dtype=out_dt, device="cuda")
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)
    assert c.layer_kernel(layer, H, W)[1] == 1                 # no split K: the staged kernels
    c.run_layer(layer, n, H, W, x, out)
    ref = deconv64(torch, ref_in, w, b) if up else conv64(torch, ref_in, w, b)
    norm = (beta + (ref * ref).view(-1, N) @ gamma.t().contiguous()).sqrt().view(ref.shape)
    ref = ref * norm if up else ref / norm
    got = out.double() / (ACT_Q if out_dt == torch.float8_e4m3fn else 1.0)
    err = float((got - ref).abs().max() / ref.abs().max())
    tol = 1e-4 if prec == FP32 else BF16_OUT_TOL if out_dt == torch.bfloat16 else FP8_OUT_TOL
    assert err < tol, f"max error / max |ref| = {err:.2e}"
    c.close()
