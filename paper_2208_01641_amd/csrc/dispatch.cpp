// Which kernel runs a layer: a choice from the layer's shape and the grids
// alone (choose_route, no device needed), and its launch.
//
// Two rules hold for every choice.  What fixes the order of a sum, the operand
// form and the K slots, depends on one image only, so a frame gives the same
// bits alone or in a batch; the kernel, its tile and its blocks depend on the
// whole batch and change no sum.
#include <algorithm>

#include "../../include/lic.h"
#include "kernels.h"

namespace lic {

// The widths that the codec's kernels are written for.  Some of them take any
// number of input channels at run time (conv_split), and would read and write
// past their tiles at others.
static bool codec_widths(const ConvShape& L)
{
    const int ci = L.cin, co = L.cop;
    switch (L.tag) {
    case LIC_GA0: return ci == 96 && (co == 128 || co == 192);
    case LIC_GA1: case LIC_GA2: case LIC_GS1: case LIC_GS2: return ci == co && (co == 128 || co == 192);
    case LIC_GS0: return (ci == 192 && co == 128) || (ci == 320 && co == 192 && L.ld == LD_I8);
    case LIC_GA3: case LIC_HA1: case LIC_HA2: case LIC_HS0: case LIC_HS1: case LIC_GS3: return ci == 128 || ci == 192;
    case LIC_HA0: return ci == 192 || (ci == 320 && L.ld == LD_F32_ABS);
    case LIC_HS2: return ci == 128 || (ci == 192 && L.ep == EP_INDEX);
    case LIC_CX: return ci == 192;
    case LIC_EP0A: case LIC_EP0N: return ci == 768;
    case LIC_EP1A: case LIC_EP1N: return ci == 640;
    case LIC_EP2A: case LIC_EP2N: return ci == 512;
    }
    return true;                                        // the distilled network: by its kernels' keys
}

namespace {

struct Grid {
    long pixels;            // of the whole batch
    int nphase;
    // blocks of nt 16-pixel tiles
    long tiles(int nt) const { return (pixels + 16 * nt - 1) / (16 * nt) * nphase; }
};

// GDN and IGDN layers behind the image layer: both operands staged in LDS, one
// or two 16-pixel tiles per wave (the same sums either way).
bool route_staged(const ConvShape& L, const ConvArgs& a, const Grid& g, ConvRoute* r)
{
    KernelKey ks = r->key;
    if (ks.dt == DT_F32) ks.dt = DT_F32X;
    ks.waves = ks.dt == DT_F32X && ks.mt == 12 ? 8 : 4;
    ks.nt = g.tiles(2) >= 1024 ? 2 : 1;
    if (!gdn_available(ks)) ks.nt = 1;
    if (!gdn_available(ks)) return false;
    r->key = ks;
    r->kernel = ConvRoute::STAGED;
    // Large grids of g_s: a tile's pixels and their halo in LDS (again the
    // same sums), 256 pixels and a phase per block.  16 x 16 or 8 x 32 pixels, whichever
    // leaves fewer tiles.  Measured against the above (us; blocks in
    // brackets): bf16 30 -> 33 [240], 52 -> 42 [416], 53 -> 43 [448], 104 -> 77
    // [960]; FP32 86 -> 91 [240], 160 -> 138 [416], 350 -> 297 [960]; e4m3 22
    // -> 23 [240], 38 -> 31 [416], 77 -> 56 [960]; 192 channels bf16 54 -> 55
    // [240], 101 -> 87 [448], e4m3 41 -> 36 [240], 74 -> 59 [448].  Just above
    // 512 blocks, where those kernels just fill the chip twice, they stay
    // ahead (FP32 176 against 183, e4m3 43 against 46 [540]).
    if (L.halo1 && L.ep == EP_IGDN && L.ld == LD_F32 && window_available(L.tag, L.cin, L.cop, ks.dt)) {
        auto blocks = [&](int tw) {
            const int th = kWindowPixels / tw;
            return (long)a.n * ((a.Hg + th - 1) / th) * ((a.Wg + tw - 1) / tw) * L.nphase;
        };
        const int tw = blocks(32) < blocks(16) ? 32 : 16;
        const long nb = blocks(tw);
        const bool twice = nb > 512 && (g.pixels + 127) / 128 * L.nphase <= 1024;
        if (nb >= (L.cop == 192 && ks.dt == DT_FP8 ? 200 : 400) && !twice) {
            r->kernel = ConvRoute::WINDOW;
            r->tw = tw;
        }
    }
    return true;
}

// Reduced-precision GDN layers with four K slots, on grids (of the whole batch)
// of enough blocks for the staged kernel: its waves keep the four sums side by
// side, so a block's weights serve 64 pixels instead of 16 or 32.
// Measured (layer call, us; blocks in brackets): e4m3 GA1 28 -> 34 [64], 37 -> 35 [96],
// 45 -> 35 [160], 54 -> 36 [240], GS1 43 -> 32 [384]; bf16 GA1 33 -> 49 [64], 41 -> 49
// [96], 45 -> 45 [160], GA2 54 -> 51 [192]; 192 channels e4m3 GA2 80 -> 50 [240], bf16
// GA1 66 -> 70 [96], 93 -> 73 [160], GA2 122 -> 75 [240].
bool route_four_sums(const ConvShape& L, const Grid& g, ConvRoute* r)
{
    KernelKey k4 = r->key;
    k4.nt = 1;
    k4.waves = 4;
    if (!gdn_available(k4) || g.tiles(4) < (L.dt == DT_FP8 ? 96 : 160)) return false;
    r->key = k4;
    r->kernel = ConvRoute::STAGED;
    return true;
}

// Split K: the K slots are in the key, the tile of a block is free (the same
// sums whatever it is): the largest that still gives the chip enough blocks.
bool route_split(const ConvShape& L, const ConvArgs& a, const Grid& g, ConvRoute* r)
{
    const bool gdn = L.ep == EP_GDN || L.ep == EP_IGDN;
    SplitKey sk{4, 1, gdn ? r->key.mt / 4 : 1, r->key.ksplit, L.ld, L.ep, L.dt};
    auto blocks = [&](int mt, int nt) { return g.tiles(nt) * (gdn ? 1 : L.cop / (16 * mt)); };
    bool two_pass = false;
    if (gdn) {
        // (FP32; layer call, us, 16- and 32-pixel tiles: GA1 at 256 x 256, four
        // images, 147 and 143 [512], GS2 at 128 x 128 68 and 68 [512], 115 and 117 [1024])
        if (blocks(4, 2) >= 512) sk.nt = 2;
        if (!split_available(sk)) sk.nt = 1;
        // The smallest FP32 GDN layers leave most of the chip idle in blocks of
        // all rows: the sums in blocks of 16 or 32 rows instead, then the normalisation in
        // place by a second launch (layer call, us; blocks of all rows in
        // brackets): GA2 49 -> 31 [4], 49 -> 31 [16], 49 -> 36 [64], 50 -> 42 [96], 52 ->
        // 51 [140]; GS1 33 -> 29 [64], 33 -> 34 [144]; 192 channels GA1 83 -> 51 [64], 88 ->
        // 76 [144], 95 -> 106 [256].  Blocks of 16 rows up to 48: 31 against 35 [16], 37
        // against 36 [64].
        const long whole = blocks(4, 1);
        if (L.dt == DT_F32 && !a.co_ld && whole <= (L.cop == 128 ? 128 : 160)) {
            const SplitKey sums{whole <= 48 ? 1 : 2, 1, 1, r->key.ksplit, L.ld, EP_NONE, DT_F32};
            if (split_available(sums)) {
                sk = sums;
                two_pass = true;
            }
        }
    } else if (L.cop % 64 == 0 && blocks(4, 2) >= (L.dt == DT_F32 ? 1024 : 320)) {
        // Measured at 720p (us; blocks in brackets): g_a's last layer 64 x 32 62
        // [360], 64 x 16 53 [720], 32 x 16 58 [1440]; the same at 470 x 834 36
        // [168], 35 [336], 31 [672]; h_a's second 31 [60], 19 [120], 14 [240],
        // 16 x 16 15 [480]; its third 31, 18, 12 [60], 10 [120]; bf16 g_a's last 18
        // [360], 21 [720].
        sk.nt = 2;
    } else if (L.cop % 64 != 0 || blocks(4, 1) < 448) {
        // (eight slots: four take at least 512 tiles of 64 x 32)
        sk.mt = L.cop % 32 == 0 && blocks(2, 1) >= 200 ? 2 : 1;
    }
    if (!split_available(sk)) return false;
    r->kernel = two_pass ? ConvRoute::TWO_PASS : ConvRoute::SPLIT;
    r->split = sk;
    r->ncog = gdn && !two_pass ? 1 : L.cop / (16 * sk.mt);
    return true;
}

}  // namespace

int choose_route(const ConvShape& L, const ConvArgs& a, long policy_pixels, ConvRoute* r, std::string* errp)
{
    const bool own = L.tag < LIC_NUM_LAYERS;            // a codec layer (else the distilled network: conv_igemm only)
    const bool gdn = L.ep == EP_GDN || L.ep == EP_IGDN;
    const Grid g{(long)a.n * a.Hg * a.Wg, L.nphase};
    *r = ConvRoute{};
    KernelKey& key = r->key;
    key = KernelKey{L.tag, L.cin, 0, 0, 0, 1, L.ld, L.ep, L.dt};
    r->ncog = 1;
    r->kernel = ConvRoute::DIRECT;
    if (gdn) {
        key.mt = L.cop / 16;
        key.nt = key.mt <= 8 ? 2 : 1;
        key.waves = 4;
        // Fewer than one wave per SIMD (1024 on the chip) from the pixel
        // grid of one image: split K over the 4 waves of a block instead,
        // unless 16-pixel groups give at least half a wave per SIMD (128
        // channels; of the e4m3 layers only GA2).  The choice sets the order
        // of the sums, so it looks at one image only and not at the batch.
        const long img_waves = (policy_pixels + 16 * key.nt - 1) / (16 * key.nt) * L.nphase;
        const long waves1 = (policy_pixels + 15) / 16 * L.nphase;
        if (L.ld != LD_RGB && img_waves < 1024 &&
            !(key.mt == 8 && waves1 >= 512 && (L.dt != DT_FP8 || L.tag == LIC_GA2)))
            key.ksplit = 4;
        if (own && L.ld == LD_RGB && L.nphase == 1 && a.kk == 5 && a.s_in == 2 && a.Wg % 32 == 0 &&
            image_available(L.cop, key.dt == DT_F32 ? DT_F32X : key.dt)) {
            if (key.dt == DT_F32) key.dt = DT_F32X;
            r->kernel = ConvRoute::IMAGE;
        } else if (own && L.ld != LD_RGB && key.ksplit == 1) {
            route_staged(L, a, g, r);
        }
    } else if (L.ep == EP_RGB) {
        // every row of the transposed convolution to 3 channels in one wave;
        // halo tiles staged per block when the taps allow
        key.mt = L.cop / 16;
        key.nt = 4;
        key.waves = 4;
        if (own && L.halo1 && L.ld == LD_F32 && a.s_out == 2 && L.cop == 16 && a.Hg % 8 == 0 && a.Wg % 32 == 0 &&
            rgb_available(L.cin, L.dt)) {
            key.ld = LD_TILE;
            r->kernel = ConvRoute::RGB;
        } else if (L.halo1 && L.ld == LD_F32) {
            KernelKey kt = key;
            kt.ld = LD_TILE;
            if (kernel_available(kt)) key = kt;
        }
    } else {
        // 64-channel x 32-pixel wave tiles; when the grid of one image gives
        // fewer than 2 waves per SIMD, split K over 4 or 8 waves of a block;
        // grids of fewer than 128 such tiles (the 24 x 40 and 12 x 20 hyper
        // layers of a 720p frame) take 16 x 16 tiles (split 8) instead, for
        // 8 times the blocks (measured: h_a's second layer 44 -> 30 us, h_s's
        // first 22 -> 16 us; the 48 x 80 layers are slower that way).  The
        // choice depends on the per-image size only, so a frame gives the
        // same bits alone or in a batch (split-K changes the summation order).
        const long tiles_big = ((policy_pixels + 31) / 32) * L.nphase * (L.cop / 64);
        key.mt = 4; key.nt = 2;
        if (L.cop % 64 != 0 || tiles_big < 128) {
            key.mt = 1; key.nt = 1; key.waves = 8; key.ksplit = 8;
        } else if (tiles_big >= 2048) {
            key.waves = 4; key.ksplit = 1;
        } else if (tiles_big * 4 >= 2048) {
            key.waves = 4; key.ksplit = 4;
        } else {
            key.waves = 8; key.ksplit = 8;
        }
        r->ncog = L.cop / (16 * key.mt);
    }
    // the image layer at 192 channels, FP32 form: split-FP32 operands
    if (own && r->kernel == ConvRoute::DIRECT && key.dt == DT_F32 && key.ksplit == 1 && gdn) {
        KernelKey kx = key;
        kx.dt = DT_F32X;
        if (kernel_available(kx)) key = kx;
    }
    if (own && key.ksplit > 1 && !(gdn && route_four_sums(L, g, r))) route_split(L, a, g, r);
    const bool split = r->kernel == ConvRoute::SPLIT || r->kernel == ConvRoute::TWO_PASS;
    const bool staged = r->kernel == ConvRoute::STAGED || r->kernel == ConvRoute::WINDOW;
    const long per_block = (long)(staged ? key.waves : key.waves / key.ksplit) * key.nt * 16;
    // halo tiles: one block per key.waves grid rows x 16 key.nt pixels
    const long tiles = split ? (g.pixels + 16 * r->split.nt - 1) / (16 * r->split.nt)
                       : key.ld == LD_TILE
                           ? (long)a.n * ((a.Hg + key.waves - 1) / key.waves) * ((a.Wg + 16 * key.nt - 1) / (16 * key.nt))
                           : (g.pixels + per_block - 1) / per_block;
    r->nblocks = tiles * L.nphase * r->ncog;
    if (r->nblocks > (1L << 30)) { *errp = "launch too large"; return LIC_E_BUDGET; }
    if (!codec_widths(L) || (r->kernel == ConvRoute::DIRECT && !kernel_available(key))) {
        *errp = "no kernel instantiated for this layer shape";
        return LIC_E_ARG;
    }
    return LIC_OK;
}

Operands layer_operands(const ConvShape& L)
{
    Operands o{};
    if (L.ep == EP_GDN || L.ep == EP_IGDN) {
        const bool direct = L.ld == LD_RGB && !image_available(L.cop, L.dt == DT_F32 ? DT_F32X : L.dt);
        o.w = direct && L.dt != DT_F32;
        o.wx = direct && L.dt == DT_F32;
        o.gsplit = direct;
        o.ws = o.gt = !direct;
        o.wt = L.ld != LD_RGB;
    } else {
        o.ws = true;
    }
    return o;
}

int launch_conv_policy(const ConvShape& L, ConvArgs& a, long policy_pixels, hipStream_t s, std::string* errp,
                       KernelKey* chosen)
{
    ConvRoute r;
    if ((long)a.n * a.Hg * a.Wg <= 0 && !chosen) return LIC_OK;
    const int rc = choose_route(L, a, policy_pixels, &r, errp);
    if (rc != LIC_OK) return rc;
    if (chosen) {
        *chosen = r.key;
        return LIC_OK;
    }
    a.ncog = r.ncog;
    a.tw = r.tw;
    const int nb = (int)r.nblocks;
    hipError_t e = hipSuccess;
    switch (r.kernel) {
    case ConvRoute::WINDOW: e = launch_window(L.tag, L.cin, L.cop, r.key.dt, a, s); break;
    case ConvRoute::IMAGE: e = launch_image(r.key.dt, a, s); break;
    case ConvRoute::RGB: e = launch_rgb(L.cin, L.dt, a, s); break;
    case ConvRoute::STAGED: e = launch_gdn(r.key, a, nb, s); break;
    case ConvRoute::SPLIT: e = launch_split(r.split, a, nb, s); break;
    case ConvRoute::TWO_PASS:
        e = launch_split(r.split, a, nb, s);
        if (e == hipSuccess) e = launch_gdn_apply(L.cop, L.ep, a, s);
        break;
    case ConvRoute::DIRECT:
        if (L.dt == DT_F32 && r.key.dt == DT_F32X) a.w = a.wx;
        e = launch_conv(r.key, a, nb, s);
        break;
    }
    if (e != hipSuccess) {
        *errp = std::string("kernel launch failed: ") + hipGetErrorString(e);
        return LIC_E_HIP;
    }
    return LIC_OK;
}

}  // namespace lic
