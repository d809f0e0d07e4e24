"""Weight blobs whose layers do not fit together: refused when a codec is made,
before anything is packed; and widths that no kernel is written for, refused
when the layer is called."""
import ctypes

import numpy as np
import pytest

import synth


def create(P, kind, N, M):
    """codec_create's status for these parameters (on a machine without a GPU a
    good blob gets as far as the device)."""
    from paper_2208_01641_amd import _lib
    blob = synth.weight_blob(P, kind, N, M)
    cfg = _lib.CodecConfig()
    _lib.lib.codec_default_config(ctypes.byref(cfg))
    cfg.kind, cfg.N, cfg.M, cfg.max_h, cfg.max_w, cfg.max_in_flight, cfg.entropy_threads = kind, N, M, 64, 64, 1, 1
    buf, h = ctypes.create_string_buffer(blob, len(blob)), ctypes.c_void_p()
    rc = _lib.lib.codec_create(ctypes.byref(cfg), buf, len(blob), ctypes.byref(h))
    if rc == 0:
        _lib.lib.codec_destroy(h)
    return rc


def widened(P, name, axis, width):
    """The same parameters with one axis of a layer's weights of another width (its bias with its output)."""
    Q = dict(P)
    shape = list(P[name + ".w"].shape)
    shape[axis] = width
    Q[name + ".w"] = np.zeros(shape, P[name + ".w"].dtype)
    if axis == (1 if name[:2] in ("gs", "hs") and name != "hs2" else 0):
        Q[name + ".b"] = np.zeros(width, P[name + ".b"].dtype)
    return Q


@pytest.mark.parametrize("kind,N,M", [(0, 128, 192), (1, 128, 192), (1, 192, 320), (2, 128, 192)])
def test_consistent_models_pass(kind, N, M):
    assert create(synth.model_params(kind, N, M), kind, N, M) in (0, -3)        # made, or no device


# (kind, layer, axis of its weights, width)
BAD = [(1, "hs0", 0, 384), (1, "hs0", 0, 192), (1, "ha0", 1, 320), (1, "ga1", 1, 192), (1, "ga2", 0, 192), (1, "ga3", 0, 320),
       (1, "gs0", 0, 320), (1, "gs2", 1, 192), (1, "gs3", 0, 192), (1, "hs2", 0, 384), (1, "ha2", 0, 192), (1, "ha1", 1, 120),
       (0, "gs0", 0, 208), (2, "cx", 1, 128), (2, "ep1", 1, 512), (2, "ep2", 1, 640), (2, "hs2", 1, 192)]


@pytest.mark.parametrize("kind,name,axis,width", BAD)
def test_layers_that_do_not_fit_are_refused(kind, name, axis, width):
    P = synth.model_params(kind, 128, 192)
    assert create(widened(P, name, axis, width), kind, 128, 192) == -8          # LIC_E_MODEL


@pytest.mark.gpu
def test_widths_without_kernels_are_refused():
    """Hyper layers of 64 channels fit together and the pools; no kernel is
    written for layers that take 64."""
    from paper_2208_01641_amd import Codec
    import torch
    N, M = 128, 192
    P = synth.model_params(1, N, M)
    for name, axes in (("ha0", (0,)), ("ha1", (0, 1)), ("ha2", (1,)), ("hs0", (1,)), ("hs1", (0, 1)), ("hs2", (1,))):
        for a in axes:
            P = widened(P, name, a, 64)
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, max_h=64, max_w=64, max_in_flight=1)
    x = torch.zeros(1 << 16, device="cuda")
    for layer in ("HA1", "HA2", "HS1", "HS2"):
        with pytest.raises(RuntimeError) as e:
            c.run_layer(layer, 1, 64, 64, x, torch.zeros(1 << 16, device="cuda"), torch.zeros(1 << 16, device="cuda"))
        assert e.value.code == -1
    for layer in ("HA0", "HS0"):
        c.run_layer(layer, 1, 64, 64, x, torch.zeros(1 << 16, device="cuda"))
    c.close()
