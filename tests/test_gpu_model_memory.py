"""A codec holds each weight only in the layouts that its kernels read."""
import numpy as np
import pytest

import synth
from gpu_util import dims

pytestmark = pytest.mark.gpu

GDN = ("ga0", "ga1", "ga2", "gs0", "gs1", "gs2")


@pytest.mark.parametrize("N,M", [(128, 192), (192, 320)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_weights_are_held_once_per_layout(prec, N, M):
    """Bytes per weight: FP32 GDN layers 6 (three bf16 parts) + 4 (split K); other
    FP32 layers 4 + 4 (row-major, for grids that need no split K, and split K); the
    reduced forms' 2 or 1 once for the GDN layers and g_s's last, twice for g_a's last
    (e4m3: chunks rounded up to 128, at most a third more).  gamma 2 or 3 bf16 parts."""
    from paper_2208_01641_amd import Codec
    P = synth.model_params(1, N, M)
    c = Codec(synth.weight_blob(P, 1, N, M), kind=1, N=N, M=M, precision=prec, max_h=64, max_w=64, max_in_flight=1)
    held = c.stats()["device_bytes"]
    c.close()
    most = 0.0
    for name in sorted({k.split(".")[0] for k in P if k.endswith(".w")}):
        n = P[name + ".w"].size * (4 / 3 if name == "gs3" else 96 / 75 if name == "ga0" else 1)   # zero rows and columns
        if name == "gs3":
            n *= 16 * 9 / (12 * 25 / 3)                        # 4 phases x 3 channels over 3 x 3 taps
        if prec == 0 or name[0] == "h":
            most += n * (10 if name in GDN else 8)
        else:
            e = 2 if prec == 1 or name in ("ga0", "gs0", "gs3") else 4 / 3
            most += n * e * (2 if name == "ga3" else 1)
        if name in GDN:
            most += N * N * 6
    d = dims(64, 64)
    pools = 4 * 4 * N * d["Hp"] * d["Wp"] + 16 * (M + N) * d["Hy"] * d["Wy"] + 4 * 6 * d["Hp"] * d["Wp"]
    assert held <= most + pools + 200_000, f"{held / 1e6:.1f} MB, at most {(most + pools) / 1e6:.1f} expected"
