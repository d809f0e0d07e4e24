"""codec_run_layer on buffers at any element: a view that starts in the middle of
an allocation gives the bytes that the same data at an aligned address gives,
and nothing beside the output is written.

The kernels' wide loads and stores want 16-byte addresses, so every layer is
run with its input one element, three elements and eight bytes further on, and
the GDN layers with their output so.  Sizes reach the split, two-pass, staged,
window and image kernels.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

LAYERS = ["GA0", "GA1", "GA2", "GA3", "GS0", "GS1", "GS2", "GS3"]
HYPER = ["HA0", "HA1", "HA2", "HS0", "HS1", "HS2"]
GDN = ("GA0", "GA1", "GA2", "GS0", "GS1", "GS2")
SIZES = [(1, 64, 64), (2, 200, 300), (1, 448, 704), (9, 320, 448)]


@pytest.mark.parametrize("kind,prec", [(1, 0), (1, 1), (1, 2), (2, 0), (2, 1)])
@pytest.mark.parametrize("n,H,W", SIZES)
def test_views_at_any_element(kind, prec, n, H, W):
    import torch

    from paper_2208_01641_amd import Codec
    N, M = 128, 192
    P = synth.model_params(kind, N, M, gamma="dense")
    c = Codec(synth.weight_blob(P, kind, N, M), kind=kind, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)
    g = torch.Generator(device="cuda")
    g.manual_seed(n * H + W)
    layers = LAYERS + HYPER if (kind, prec) == (1, 0) else LAYERS if kind == 1 else ["GS0", "HA0", "HS2", "CX", "EP0A", "EP1N"]
    for layer in layers:
        bi, bo, ba = c.layer_bytes(layer, n, H, W)
        if layer == "HS0" or (layer == "GS0" and kind == 1):
            x = torch.randint(-9, 10, (bi,), dtype=torch.int8, device="cuda", generator=g)
        elif prec == 0 or layer == "GA0" or layer[0] in "HCE":
            x = torch.randn(bi // 4, device="cuda", generator=g)
        elif prec == 1 or layer in ("GS0", "GS3"):
            x = torch.randn(bi // 2, device="cuda", generator=g).to(torch.bfloat16)
        else:
            x = (8 * torch.randn(bi, device="cuda", generator=g)).to(torch.float8_e4m3fn)
        esz = x.element_size()
        want, waux = (torch.zeros(max(b, 1), dtype=torch.uint8, device="cuda") for b in (bo, ba))
        c.run_layer(layer, n, H, W, x, want, waux if ba else None)
        for shift in sorted({esz, 3 * esz, 8}):
            room = torch.zeros(bi + 32, dtype=torch.uint8, device="cuda")
            view = room[shift:shift + bi]
            view.copy_(x.view(torch.uint8))
            assert view.data_ptr() % 16 == shift
            got, aux = torch.zeros_like(want), torch.zeros_like(waux)
            c.run_layer(layer, n, H, W, view, got, aux if ba else None)
            assert torch.equal(got, want) and torch.equal(aux, waux), f"{layer}: input {shift} bytes on"
            if layer in GDN:
                room = torch.full((bo + 32,), 77, dtype=torch.uint8, device="cuda")
                c.run_layer(layer, n, H, W, view, room[shift:shift + bo])
                assert torch.equal(room[shift:shift + bo], want), f"{layer}: output {shift} bytes on"
                assert bool((room[:shift] == 77).all()) and bool((room[shift + bo:] == 77).all())
    c.close()


def test_frames_of_a_batch_at_any_float():
    """Frames whose bytes are no multiple of 16: each starts at another float."""
    import torch

    from paper_2208_01641_amd import Codec
    N, M, n, H, W = 128, 192, 3, 65, 67
    P = synth.model_params(1, N, M, gamma="dense")
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, max_h=H, max_w=W, max_in_flight=2)
    x = synth.frames_sinusoid_torch(H, W, range(n))
    assert {x[i].data_ptr() % 16 for i in range(n)} != {0}
    out = torch.empty_like(x)
    streams = c.encode_decode(x, out)
    for i in range(n):
        one = x[i:i + 1].clone()
        back = torch.empty_like(one)
        assert c.encode_decode(one, back) == [streams[i]]
        assert np.array_equal(back.cpu().numpy(), out[i:i + 1].cpu().numpy())
    c.close()
