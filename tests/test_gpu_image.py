"""The two layers at the image end, g_a's first and g_s's last: whole tensors
against the same layer in float64.

Sizes: one 32-pixel tile a row, fewer tiles than CUs, ragged widths and
heights (zero padding, crop), several images, and grids with more tiles than
one round of waves.  The reference takes the operands as the form rounds them;
what is left is FP32 accumulation (1e-4 of max |ref|) and one rounding of a
stored bf16 (2^-8) or e4m3 (2^-4) output.
"""
import numpy as np
import pytest

import synth
from gpu_util import dims
from test_gpu_fp8 import FP8_OUT_TOL
from test_gpu_precision import BF16_OUT_TOL, bf16
from test_gpu_staged import ACT_Q, conv64, deconv64

pytestmark = pytest.mark.gpu

SIZES = [(1, 64, 64), (3, 65, 333), (1, 448, 640), (2, 200, 1000)]


@pytest.mark.parametrize("n,H,W", SIZES)
@pytest.mark.parametrize("N,M", [(128, 192), (192, 320)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_image_layers(prec, N, M, n, H, W):
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    Hp, Wp = d["Hp"], d["Wp"]
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)
    g = torch.Generator(device="cuda")
    g.manual_seed(H * W + n)

    def params(name, *keys):
        w = P[name + ".w"] if prec == 0 else bf16(P[name + ".w"])
        return [torch.from_numpy(np.asarray(t, np.float64)).cuda() for t in [w] + [P[name + k] for k in keys]]

    # g_a's first layer: NCHW image, bf16 operands in the reduced forms
    x = torch.rand((n, 3, H, W), device="cuda", generator=g)
    out_dt = [torch.float32, torch.bfloat16, torch.float8_e4m3fn][prec]
    out = torch.empty((n, Hp // 2, Wp // 2, N), dtype=out_dt, device="cuda")
    c.run_layer("GA0", n, H, W, x, out)
    w, b, beta, gamma = params("ga0", ".b", ".beta", ".gamma")
    xr = (x if prec == 0 else x.to(torch.bfloat16)).double()
    xr = torch.nn.functional.pad(xr, (0, Wp - W, 0, Hp - H)).permute(0, 2, 3, 1).contiguous()
    ref = conv64(torch, xr, w, b)
    ref = ref / (beta + (ref * ref).view(-1, N) @ gamma.t().contiguous()).sqrt().view(ref.shape)
    got = out.double() / (ACT_Q if prec == 2 else 1.0)
    err = float((got - ref).abs().max() / ref.abs().max())
    assert err < (1e-4, BF16_OUT_TOL, FP8_OUT_TOL)[prec], f"GA0: {err:.2e}"

    # g_s's last layer: pre-clamp image on the padded size, clamped and cropped image
    y = torch.randn((n, Hp // 2, Wp // 2, N), device="cuda", generator=g)
    y = y if prec == 0 else y.to(torch.bfloat16)
    img = torch.empty((n, 3, H, W), device="cuda")
    pre = torch.empty((n, 3, Hp, Wp), device="cuda")
    c.run_layer("GS3", n, H, W, y, img, pre)
    w, b = params("gs3", ".b")
    ref = deconv64(torch, y.double(), w, b).permute(0, 3, 1, 2)
    err = float((pre.double() - ref).abs().max() / ref.abs().max())
    assert err < 1e-4, f"GS3: {err:.2e}"
    assert torch.equal(img, pre[:, :, :H, :W].clamp(0.0, 1.0))
    img.zero_()
    c.run_layer("GS3", n, H, W, y, img)
    assert torch.equal(img, pre[:, :, :H, :W].clamp(0.0, 1.0))
    c.close()


@pytest.mark.parametrize("n,H,W", SIZES)
@pytest.mark.parametrize("N,M", [(128, 192), (192, 320)])
def test_output_layer_fp32_error(N, M, n, H, W):
    """g_s's FP32 output layer (split operands) against float64, in the 2-norm: each
    of up to 54 sums rounds once more (2^-24 sqrt(54) = 4.4e-7, twice that for what
    partial sums exceed the result by); one order of part products left out
    would give 2^-17 = 7.6e-6."""
    import torch

    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M, gamma="dense")
    d = dims(H, W)
    g = torch.Generator(device="cuda")
    g.manual_seed(H + W + n)
    x = torch.randn((n, d["Hp"] // 2, d["Wp"] // 2, N), device="cuda", generator=g)
    img = torch.empty((n, 3, H, W), device="cuda")
    pre = torch.empty((n, 3, d["Hp"], d["Wp"]), device="cuda")
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, max_h=64, max_w=64, max_in_flight=1)
    c.run_layer("GS3", n, H, W, x, img, pre)
    w, b = (torch.from_numpy(np.asarray(P["gs3" + k], np.float64)).cuda() for k in (".w", ".b"))
    ref = deconv64(torch, x.double(), w, b).permute(0, 3, 1, 2)
    err = float((pre.double() - ref).norm() / ref.norm())
    assert err < 1e-6, f"{err:.2e}"
    assert torch.equal(img, pre[:, :, :H, :W].clamp(0.0, 1.0))
    c.close()
