"""g_s's GDN layers on the kernels that hold a pixel tile and its halo in LDS
(large grids, batches): each image of a batch against the same image alone,
whose grid is too small for them, and one image against float64.

Neither the tile nor the batch changes a sum, so the images of a batch are
the same bytes.  Grids whose last tile is not full in rows, columns or both,
tiles of 16 and of 32 columns, and GDN and 1DN.  The float64 reference takes
the operands as the form rounds them (tolerances of test_gpu_staged).
"""
import numpy as np
import pytest

import synth
from gpu_util import dims
from test_gpu_fp8 import FP8_OUT_TOL, w_fp8
from test_gpu_precision import BF16_OUT_TOL, bf16
from test_gpu_staged import ACT_Q, deconv64

pytestmark = pytest.mark.gpu

FP32, BF16, FP8 = 0, 1, 2
# (precision, layer, N, M, n, H, W, norm)
CASES = [
    (prec, layer, 128, 192, n, H, W, 0) for prec in (FP32, BF16)
    for layer, n, H, W in (("GS1", 9, 448, 320), ("GS1", 12, 192, 704), ("GS2", 9, 256, 192))
] + [
    (FP32, "GS2", 128, 192, 9, 256, 192, 1), (BF16, "GS1", 128, 192, 7, 320, 768, 1),
    (FP8, "GS1", 128, 192, 3, 576, 960, 0), (FP8, "GS2", 128, 192, 9, 320, 448, 0), (FP8, "GS2", 128, 192, 9, 320, 448, 1),
    (BF16, "GS1", 192, 320, 5, 448, 704, 0), (BF16, "GS1", 192, 320, 5, 832, 320, 0), (BF16, "GS2", 192, 320, 7, 256, 320, 1),
    (FP8, "GS1", 192, 320, 6, 576, 512, 0), (FP8, "GS2", 192, 320, 3, 320, 448, 0),
]


@pytest.mark.parametrize("prec,layer,N,M,n,H,W,norm", CASES)
def test_window_layer(prec, layer, N, M, n, H, W, norm):
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    den = {"GS1": 8, "GS2": 4}[layer]
    hi, wi = d["Hp"] // den, d["Wp"] // den
    g = torch.Generator(device="cuda")
    g.manual_seed(hi * wi + n)
    x = torch.randn((n, hi, wi, N), device="cuda", generator=g)
    x = (ACT_Q * x).to(torch.float8_e4m3fn) if prec == FP8 else x.to(torch.bfloat16) if prec == BF16 else x
    out_dt = torch.float32 if prec == FP32 else torch.bfloat16 if prec == BF16 or layer == "GS2" else torch.float8_e4m3fn
    out = torch.empty((n, 2 * hi, 2 * wi, N), dtype=out_dt, device="cuda")
    alone = torch.empty((1, 2 * hi, 2 * wi, N), dtype=out_dt, device="cuda")
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1, norm=norm)
    assert c.layer_kernel(layer, H, W)[1] == 1                 # no split K
    c.run_layer(layer, n, H, W, x, out)
    for i in range(n):
        c.run_layer(layer, 1, H, W, x[i:i + 1].contiguous(), alone)
        assert torch.equal(out[i].view(torch.uint8), alone[0].view(torch.uint8)), f"image {i} of {n} differs"

    name = layer.lower()
    w = P[name + ".w"]
    w = w if prec == FP32 else bf16(w) if prec == BF16 else w_fp8(w, "deconv")
    w, b, beta, gamma = (torch.from_numpy(np.asarray(t, np.float64)).cuda()
                         for t in (w, P[name + ".b"], P[name + ".beta"], P[name + ".gamma"]))
    ref = deconv64(torch, x[n - 1:].double() / (ACT_Q if prec == FP8 else 1.0), w, b)
    r = ref.abs() if norm else ref * ref
    r = (beta + r.view(-1, N) @ gamma.t().contiguous()).view(ref.shape)
    ref = ref * (r if norm else r.sqrt())
    got = out[n - 1:].double() / (ACT_Q if out_dt == torch.float8_e4m3fn else 1.0)
    if out_dt == torch.float8_e4m3fn:
        ref = ref.clamp(-448 / ACT_Q, 448 / ACT_Q)
    err = float((got - ref).abs().max() / ref.abs().max())
    tol = 1e-4 if prec == FP32 else BF16_OUT_TOL if out_dt == torch.bfloat16 else FP8_OUT_TOL
    assert err < tol, f"max error / max |ref| = {err:.2e}"
    c.close()
