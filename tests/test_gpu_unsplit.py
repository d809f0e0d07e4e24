"""Layers of frames so large that K is not split (conv_igemm), which read the
weights in the split-K kernels' order, and the device memory that a second
layout of them would take (a budget that was enough would refuse the codec).

Against float64 on operands as the form rounds them: what is left is FP32
accumulation of up to 25 x 320 products (1e-4 of max |ref|).
"""
import numpy as np
import pytest

import oracle
import synth
from route_util import GDN, MODELS
from test_gpu_routes import FP32, activations, codec, grids, reference
from test_gpu_split import conv3

pytestmark = pytest.mark.gpu

LAYERS = [(kind, N, M, p, layer) for kind, N, M, p, layers in MODELS for layer in layers if layer not in GDN and layer != "GS3"] + \
         [(2, 128, 192, 0, layer) for layer in ("EP0N", "EP1N", "EP2N")]


def unsplit_size(kind, N, M, prec, layer):
    """The smallest square frame (plus one block of columns) whose K is not split."""
    from paper_2208_01641_amd.codec import layer_route
    for side in range(1024, 16384, 64):
        r = layer_route(layer, 1, side, side + 64, kind, N, M, prec)
        if r["ksplit"] == 1:
            assert r["kernel"] == "direct"
            return side, side + 64
    raise AssertionError("no size with unsplit K")


@pytest.mark.parametrize("kind,N,M,prec,layer", LAYERS)
def test_unsplit_layer(kind, N, M, prec, layer):
    import torch
    P = synth.model_params(kind, N, M, gamma="dense")
    H, W = unsplit_size(kind, N, M, prec, layer)
    c = codec(kind, N, M, prec, P)
    hi, wi, ho, wo = grids(layer, H, W)
    ep = layer[:2] == "EP"
    ci = {"HA0": M, "CX": M, "EP0": 4 * M, "EP1": 640, "EP2": 512}.get(layer[:3], N)
    x, value = activations(torch, kind, prec, layer, (1, hi, wi, ci), H)
    par = (torch.arange(ho)[:, None] + torch.arange(wo)[None]).cuda() % 2
    if layer == "CX":
        w = torch.from_numpy(P["cx.w"] * oracle.context_mask()).double().cuda()
        xp = torch.nn.functional.pad(x.double(), (0, 0, 2, 2, 2, 2))
        ref = torch.from_numpy(np.asarray(P["cx.b"], np.float64)).cuda().expand(hi * wi, -1).clone()
        for u, v in zip(*np.nonzero(oracle.context_mask())):
            ref += xp[:, u:u + hi, v:v + wi].reshape(-1, M) @ w[:, :, u, v].t().contiguous()
        out = torch.full((hi, wi, 4 * M), 7.0, device="cuda")
        c.run_layer(layer, 1, H, W, x, out)
        ref = ref.view(hi, wi, 2 * M)[par == 1]
        assert bool((out[..., :2 * M] == 7.0).all()) and bool((out[par == 0] == 7.0).all())
        got = out[par == 1][:, 2 * M:]
    elif ep:
        part = 0 if layer[3] == "A" else 1
        w, b = (torch.from_numpy(np.asarray(P[layer[:3].lower() + k], np.float64)).cuda() for k in (".w", ".b"))
        ref = (x.double().view(-1, ci) @ w[:, :, 0, 0].t().contiguous() + b).view(hi, wi, -1)[par == part]
        if layer[2] == "2":                               # rows: means, then scales; the decoder's outputs
            idx = torch.zeros((2, hi, wi // 2, M), dtype=torch.uint8, device="cuda")
            mean = torch.zeros((2, hi, wi // 2, M), device="cuda")
            c.run_layer(layer, 1, H, W, x, idx, None, None, mean)
            assert int((mean[1 - part] != 0).sum()) == 0 and int((idx[1 - part] != 0).sum()) == 0
            got = mean[part].view(-1, M)
            s = ref[:, M:].cpu().numpy()
            table = oracle.scale_index_f32(s.astype(np.float32), 1).reshape(s.shape)
            assert float((idx[part].view(-1, M).cpu().numpy() != table).mean()) < 1e-4
            ref = ref[:, :M]
        else:
            out = torch.full((hi, wi, b.numel()), 7.0, device="cuda")
            c.run_layer(layer, 1, H, W, x, out)
            assert bool((out[par != part] == 7.0).all())
            got, ref = out[par == part], ref.clamp(min=0.0)
    elif layer == "HS2" and kind == 2:
        out = torch.full((1, hi, wi, 4 * M), 7.0, device="cuda")
        c.run_layer(layer, 1, H, W, x, out)
        w, b = (torch.from_numpy(np.asarray(P["hs2" + k], np.float64)).cuda() for k in (".w", ".b"))
        assert bool((out[..., 2 * M:] == 7.0).all())
        got, ref = out[..., :2 * M], conv3(torch, x.double(), w, b)
    else:
        co = M if layer in ("GA3", "HS2") else N
        ref = reference(torch, c, P, prec if layer == "GA3" else FP32, layer, kind, N, value(x))
        val = torch.zeros((1, ho, wo, co), device="cuda")
        if layer == "HS2":
            idx = torch.zeros((1, ho, wo, co), dtype=torch.uint8, device="cuda")
            c.run_layer(layer, 1, H, W, x, idx, val)
            v = val.cpu().numpy()
            assert np.array_equal(idx.cpu().numpy(), oracle.scale_index_f32(v, 1).reshape(v.shape))
        elif layer in ("GA3", "HA2"):
            sym = torch.zeros((1, ho, wo, co), dtype=torch.int8, device="cuda")
            c.run_layer(layer, 1, H, W, x, val, sym)
            mu = c.medians() if layer == "HA2" else np.float32(0)
            assert np.array_equal(sym.cpu().numpy(), np.clip(np.rint(val.cpu().numpy() - mu), -64, 64).astype(np.int8))
        else:
            c.run_layer(layer, 1, H, W, x, val)
        got = val
    c.close()
    err = float((got.double() - ref).abs().max() / ref.abs().max())
    assert err < 1e-4, f"{layer} at {H} x {W}: {err:.2e}"


#: (kind, N, M): MB of a codec of 64 x 64 frames, one in flight, by form, where every weight is held once
#: (FP32 GDN layers: as FP32 and as three bf16 parts; entropy parameters: once for each checkerboard set)
BUDGET = {(0, 128, 192): (27.3, 7.9, 5.6), (1, 128, 192): (35.6, 16.2, 14.0), (1, 192, 320): (81.4, 36.3, 31.1),
          (2, 128, 192): (60.1, 40.7, 38.5)}


@pytest.mark.parametrize("kind,N,M", list(BUDGET))
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_a_budget_without_room_for_second_layouts_is_enough(prec, kind, N, M):
    from paper_2208_01641_amd import Codec
    P = synth.model_params(kind, N, M)
    Codec(synth.weight_blob(P, kind, N, M), kind=kind, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1,
          hbm_budget_bytes=int(1e6 * BUDGET[kind, N, M][prec])).close()
