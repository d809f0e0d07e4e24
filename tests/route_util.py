"""Which kernel each layer takes at which size (host arithmetic), for the tests
that run them."""
import functools

from paper_2208_01641_amd.codec import layer_route

TRANSFORM = ["GA0", "GA1", "GA2", "GA3", "GS0", "GS1", "GS2", "GS3"]
GDN = ("GA0", "GA1", "GA2", "GS0", "GS1", "GS2")
HYPER = ["HA0", "HA1", "HA2", "HS0", "HS1", "HS2"]
CONTEXT = ["CX", "EP0A", "EP1A", "EP2A"]
#: (kind, N, M, precision, layers): the codec's models and forms (h_a, h_s and the context layers: FP32 in each)
MODELS = [(1, N, M, p, TRANSFORM + (HYPER if p == 0 else [])) for N, M in ((128, 192), (192, 320)) for p in (0, 1, 2)] + \
         [(2, 128, 192, 0, CONTEXT + ["HA0", "HS2", "GS0"]), (2, 128, 192, 1, ["GS0"]), (2, 128, 192, 2, ["GS0"])]
SIDES = [64 * k for k in (1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 17, 20, 30, 34)]
BATCHES = (1, 2, 3, 5, 9, 16, 33)
PIXELS = 5_000_000


def tile(r):
    return r["kernel"], r["form"], r["ksplit"], r["mt"], r["nt"], r["waves"], r["tw"]


@functools.lru_cache(maxsize=None)
def routes(kind, N, M, precision, layer):
    """{tile: (n, H, W)} of the smallest batch that takes it, up to PIXELS."""
    sizes = sorted((n * h * w, n, h, w) for n in BATCHES for h in SIDES for w in SIDES if n * h * w <= PIXELS)
    got = {}
    for _, n, h, w in sizes:
        got.setdefault(tile(layer_route(layer, n, h, w, kind, N, M, precision)), (n, h, w))
    return got
