// IGDN layers of g_s on large grids (transposed convolutions as stride-1
// phases, every tap within one pixel): the staged kernel of gdn_kernels.hip
// with the pixels of a tile and its one-pixel halo held in LDS.
//
// What bounds the staged kernel there: every tap stages its pixels anew (22
// bytes a clock, the window's rows missing L1), and a wave's weight fragments
// serve two pixel tiles.  Here a block of 256 pixels and one phase loads each
// 32-channel slice of its window once, one slice ahead (e4m3, whose chunks run
// through the channels of a tap before the next tap: every channel at the
// start), and a tap is an offset in LDS.  That leaves room for four pixel tiles a
// wave at 128 channels (half the fragment reads; the GDN contraction takes
// two at a time, so the registers still allow two waves per SIMD) in the reduced
// forms; split FP32 and 192 channels take two tiles and blocks of 8 waves, one
// per CU.  Weights come through the ring as before, and a step reads the
// next chunk's first fragments before its barrier.
//
// The products, their order and the order of the channels and taps are those
// of the staged kernel, so the results are the same bits.
//
// Measured against the staged kernel (kernel time, us): 720p GS2 bf16 104 ->
// 77, e4m3 77 -> 56, split FP32 350 -> 297; four 1080p frames at 192 channels bf16
// 1450 -> 1385, e4m3 1080 -> 960.  What is left at 720p bf16: 3.7 us of first
// loads, 7.5 to 11 of GDN and 3 of stores in a block of 30 to 43 us, which the
// CU's other block hides only in part; its K loop runs at 0.69 us a step of
// two blocks, 0.54 at the rate that the matrix cores hold under this load.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/lic.h"
#include "conv_args.h"
#include "gdn_finish.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

template <int TAG, int CIN, int MT, int NT, int NG, int WAVES, int ST, int DT>
__global__ void __launch_bounds__(64 * WAVES, 2) gdn_window(ConvArgs a)
{
    using Elem = typename Prec<DT>::Elem;
    static_assert(DT == DT_F32X || DT == DT_BF16 || DT == DT_FP8, "matrix-core forms");
    constexpr int KCH = Prec<DT>::KCH;
    constexpr int SUB = DT == DT_F32X ? 3 : DT == DT_FP8 ? 2 : 1;  // 1 KB weight fragments per 16 rows and chunk
    constexpr int ESZ = (int)sizeof(Elem);
    constexpr int PX = WAVES * NT * 16;                            // pixels of a block's tile
    static_assert(PX == kWindowPixels, "16 x 16 or 8 x 32 pixels");
    constexpr int WPX = 10 * 34;                                   // pixels of the larger window
    // the window: every channel (e4m3, whose chunks walk (tap, channel)), or
    // one 32-channel slice in each of two buffers
    constexpr bool WHOLE = DT == DT_FP8;
    constexpr int RB = WHOLE ? CIN * ESZ : KCH * ESZ;              // bytes of a window pixel
    constexpr int PP = RB / 16;                                    // 16-byte pieces of it
    static_assert(PP == 4 || PP == 8 || PP == 12, "swizzles below");
    constexpr int NI = (WPX * PP + 63) / 64;                       // loads of a window
    constexpr int WL = (NI + WAVES - 1) / WAVES;                   // of a wave
    constexpr int WBW = NI * 256;                                  // words of a window
    constexpr int NWB = WHOLE ? 1 : 2;
    constexpr int AP = MT * SUB;                                   // weight fragments (KB) per chunk
    constexpr int AW = (AP + WAVES - 1) / WAVES;                   // loads of them per wave (past the end: the last again)
    constexpr int STW = AP * 256;
    constexpr int RINGW = NWB * WBW + ST * STW;
    constexpr int GAMW = MT * (DT == DT_F32X ? 3 : 2) * 256 * (MT / 2);
    constexpr int OUTW = gdn_out_words(MT, WAVES, DT);
    constexpr int SMW = RINGW > GAMW ? (RINGW > OUTW ? RINGW : OUTW) : (GAMW > OUTW ? GAMW : OUTW);
    constexpr int CO = MT * 16;
    static_assert((SMW + 3 * CO) * 4 <= (WAVES == 4 ? 81920 : 163840), "two waves per SIMD");
    __shared__ __attribute__((aligned(16))) uint32_t smem[SMW + 3 * CO];
    float* const cst = reinterpret_cast<float*>(smem + SMW);       // bias, beta, e4m3 scales
    uint32_t* const ring = smem + NWB * WBW;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    // block -> (tile, phase): an XCD has a contiguous range of tiles and goes
    // through them phase by phase, the one with the most taps first (the phases
    // of a tile in turn: FP32 298 -> 352 us, bf16 77 -> 84)
    const int TW = a.tw, TH = PX / TW;
    const int ty_n = (a.Hg + TH - 1) / TH, tx_n = (a.Wg + TW - 1) / TW;
    const int T = a.n * ty_n * tx_n, Tx = (T + 7) >> 3;
    const int phase = (int)(blockIdx.x >> 3) / Tx;
    const int tile = (int)(blockIdx.x & 7) * Tx + (int)(blockIdx.x >> 3) - phase * Tx;
    if (tile >= T) return;
    const int im = tile / (ty_n * tx_n), tr = tile - im * (ty_n * tx_n);
    const int y0 = tr / tx_n * TH, x0 = (tr - tr / tx_n * tx_n) * TW;
    const int WP = TW + 2;

    // 16-byte pieces of a window pixel are rotated by its column, so that the
    // eight neighbouring pixels x two lane groups of a b128 read hit distinct
    // banks
    auto rot = [](int wx) __attribute__((always_inline)) {
        return PP == 4 ? (wx >> 1) & 3 : PP == 8 ? ((wx >> 1) & 1) | (((wx >> 2) & 1) << 2) : (wx >> 2) & 1;
    };
    const uint8_t* const in0 = static_cast<const uint8_t*>(a.in) +
                               (((long)im * a.Hin + y0 - 1) * a.Win + x0 - 1) * (long)(CIN * ESZ);
    const int wpieces = (TH + 2) * WP * PP, ni = (wpieces + 63) >> 6;
    uint32_t woff[WL];
#pragma unroll
    for (int i = 0; i < WL; ++i) {
        const int q = min(i * WAVES + wave, ni - 1) * 64 + lane;
        const int w = q / PP, slot = q - w * PP;
        const int wy = w / WP, wx = w - wy * WP;
        const bool ok = q < wpieces && (unsigned)(y0 - 1 + wy) < (unsigned)a.Hin && (unsigned)(x0 - 1 + wx) < (unsigned)a.Win;
        woff[i] = ok ? (uint32_t)((wy * a.Win + wx) * (CIN * ESZ) + (slot ^ rot(wx)) * 16) : 0xffffffffu;
    }
    auto issue_window = [&](int s) __attribute__((always_inline)) {
        const Buf b = make_buf(in0 + s * RB);
        uint32_t* const d = smem + (WHOLE ? 0 : (s & 1) * WBW);
#pragma unroll
        for (int i = 0; i < WL; ++i) buf_load_lds(b, d + min(i * WAVES + wave, ni - 1) * 256, woff[i], 0);
    };
    issue_window(0);

    const PhaseDesc* __restrict__ ph = a.ph + phase;
    const int ntaps = ph->ntaps;
    // lane t keeps tap t's offset in the window (pixels) and its dx
    const int tdy = lane < ntaps ? (int)ph->dy[lane] : 0, tdx = lane < ntaps ? (int)ph->dx[lane] : 0;
    const int tapv = (((tdy + 1) * WP + tdx + 1) << 8) | (tdx + 1);
    const Buf wbuf = make_buf(static_cast<const uint8_t*>(a.wt) + ph->wtoff * (DT == DT_F32X ? 6 : (int)sizeof(typename Prec<DT>::WElem)));
    int i_k = 0, i_st = 0;
    auto issue = [&]() __attribute__((always_inline)) {
        uint32_t* const st = ring + i_st * STW;
#pragma unroll
        for (int u = 0; u < AW; ++u) {
            const int f = AP % WAVES == 0 ? wave * AW + u : min(wave * AW + u, AP - 1);
            buf_load_lds(wbuf, st + f * 256, lane * 16, (i_k * AP + f) * 1024);
        }
        ++i_k;
        if (++i_st == ST) i_st = 0;
    };
#pragma unroll
    for (int j = 0; j < ST - 1; ++j) issue();
    for (int c = threadIdx.x; c < CO; c += 64 * WAVES) {
        cst[c] = a.bias[c];
        cst[CO + c] = a.beta[c];
        if constexpr (DT == DT_FP8) cst[2 * CO + c] = a.rscale[c];
    }

    constexpr int NS = WHOLE ? 1 : CIN / KCH;                      // slices
    const int nk = DT == DT_FP8 ? (ntaps * CIN + KCH - 1) / KCH : ntaps * NS;
    int noff[NT];                                                  // bytes from the tile's first pixel to tile nt's
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int q = wave * NT + nt;
        noff[nt] = (TW == 16 ? q * WP : (q >> 1) * WP + (q & 1) * 16) * RB;
    }
    // The fragments of the next chunk are read ahead of its barrier (AHEAD,
    // which takes a third stage): the pixels' before the last PF rows of
    // weights, and the first PF of those in the place of the last.
    constexpr bool AHEAD = ST >= 3;
    constexpr int PF = DT == DT_F32X ? 2 : 4;                      // weight fragments held
    static_assert(MT % PF == 0, "fragment slots");
    u32x4 Bl[NT], Bh[NT], A[PF][SUB];
    Split3 Bx[NT];
    int r_t = 0, r_s = 0, r_k = 0, r_st = 0;                       // chunk whose fragments are read next
    auto readA = [&](int mt) __attribute__((always_inline)) {
        const uint32_t* const as = ring + r_st * STW + lane * 4;
#pragma unroll
        for (int g = 0; g < SUB; ++g) A[mt % PF][g] = *reinterpret_cast<const u32x4*>(as + (mt * SUB + g) * 256);
    };
    auto readB = [&]() __attribute__((always_inline)) {
        const uint8_t* bb = reinterpret_cast<const uint8_t*>(smem) + (WHOLE ? 0 : (r_s & 1) * (WBW * 4));
        int ba;                                                    // the lane's bytes in the window
        if constexpr (WHOLE) {
            const int f0 = r_k * KCH, tA = f0 / CIN, c = f0 - tA * CIN + kg * 32;
            int tv = __builtin_amdgcn_readlane(tapv, min(tA, ntaps - 1)), cc = c;
            if constexpr (CIN % KCH != 0) {
                const int tv2 = __builtin_amdgcn_readlane(tapv, min(tA + 1, ntaps - 1));
                tv = c >= CIN ? tv2 : tv;
                cc = c >= CIN ? c - CIN : c;
            }
            ba = ((tv >> 8) + l16) * RB + (((cc >> 4) ^ rot((tv & 255) + l16)) << 4);
        } else {
            const int tv = __builtin_amdgcn_readlane(tapv, r_t);
            const int piece = PP == 4 ? kg : 2 * kg;
            ba = ((tv >> 8) + l16) * RB + ((piece ^ rot((tv & 255) + l16)) << 4);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            Bl[nt] = *reinterpret_cast<const u32x4*>(bb + (ba + noff[nt]));
            if constexpr (PP > 4) Bh[nt] = *reinterpret_cast<const u32x4*>(bb + ((ba ^ 16) + noff[nt]));
        }
    };
    auto next = [&]() __attribute__((always_inline)) {
        ++r_k;
        if (++r_t == ntaps) {
            r_t = 0;
            ++r_s;
        }
        if (++r_st == ST) r_st = 0;
    };
    auto split = [&](int nt) __attribute__((always_inline)) {
        const f4 lo = __builtin_bit_cast(f4, Bl[nt]), hi = __builtin_bit_cast(f4, Bh[nt]);
        const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return split3(v);
    };

    f4 acc[MT][NT];
    auto step = [&](auto more, int c_t, int c_s) __attribute__((always_inline)) {
        u32x4 Cl[NT], Ch[NT];
        Split3 Cx[NT];
        if constexpr (!AHEAD) {
            readB();
#pragma unroll
            for (int mt = 0; mt < PF; ++mt) readA(mt);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            Cl[nt] = Bl[nt];
            Ch[nt] = Bh[nt];
            if constexpr (DT == DT_F32X) Cx[nt] = AHEAD ? Bx[nt] : split(nt);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(more)::value) {
            issue();
            if (!WHOLE && c_t == 0 && c_s + 1 < NS) issue_window(c_s + 1);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const u32x4(&W)[SUB] = A[mt % PF];
            if constexpr (DT == DT_F32X) {
                // the six part products, smallest first
                constexpr int pa[6] = {0, 1, 2, 0, 1, 0}, pbx[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
                for (int s = 0; s < 6; ++s)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[pa[s]]), Cx[nt].p[pbx[s]],
                                                                              acc[mt][nt], 0, 0, 0);
            } else if constexpr (DT == DT_BF16) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[0]),
                                                                          __builtin_bit_cast(bf16x8, Cl[nt]), acc[mt][nt], 0, 0, 0);
            } else {
                auto cat = [](const u32x4& lo, const u32x4& hi) {
                    return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
                };
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        cat(W[0], W[SUB - 1]), cat(Cl[nt], Ch[nt]), acc[mt][nt], 0, 0, 0, kE8M0One, 0, kE8M0One);
            }
            if (mt + PF < MT) {
                readA(mt + PF);
                if (AHEAD && mt + PF == MT - 1) {
                    next();
                    readB();
                }
            } else if (AHEAD) {
                readA(mt + PF - MT);
                if constexpr (DT == DT_F32X)
                    if (mt + NT >= MT) Bx[mt + NT - MT] = split(mt + NT - MT);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!AHEAD) next();
    };

    // Step k issues chunk k + ST - 1 into the stage of chunk k - 1, and the next
    // slice's window in a slice's first step, after that step's weights.
    // Step k needs chunk k (AHEAD: k + 1) and waits with the later ones in
    // flight, and a window until a younger chunk is needed; it has landed
    // when its first fragments are read, at least three steps on.
    static_assert(ST >= 2 && ST <= 4, "a phase has at least four taps");
    constexpr int LATER = (AHEAD ? ST - 3 : ST - 2) * AW;
    wait_vm<0>();                                       // (the compiler then adds no waits of its own to the loop)
    lds_barrier();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f4 b = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (DT != DT_FP8) b = *reinterpret_cast<const f4*>(cst + mt * 16 + kg * 4);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = b;
    }
    if constexpr (AHEAD) {
        readB();
#pragma unroll
        for (int mt = 0; mt < PF; ++mt) readA(mt);
        if constexpr (DT == DT_F32X) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) Bx[nt] = split(nt);
        }
    }
    int k = 0, c_t = 0, c_s = 0;
    for (; k + ST - 1 < nk; ++k) {
        if (!WHOLE && ST > 2 && c_t >= 1 && c_t <= ST - 2 && c_s + 1 < NS) wait_vm<LATER + WL>();
        else wait_vm<LATER>();
        lds_barrier();
        step(std::true_type{}, c_t, c_s);
        if (++c_t == ntaps) {
            c_t = 0;
            ++c_s;
        }
    }
    for (; k < nk; ++k) {
        wait_vm<0>();
        lds_barrier();
        step(std::false_type{}, 0, 0);
    }
    lds_barrier();                                      // window and ring are free

    const long oc = a.co_ld ? a.co_ld : a.Co;
    gdn_finish<MT, NT, NG, WAVES, SMW, EP_IGDN, DT, true>(a, cst, acc, smem, lane, wave, [&](int nt) __attribute__((always_inline)) {
        const int q = wave * NT + nt;
        const int y = y0 + (TW == 16 ? q : q >> 1), x = x0 + (TW == 16 ? 0 : (q & 1) * 16) + l16;
        return y < a.Hg && x < a.Wg
                   ? (((long)im * a.Hout + y * a.s_out + ph->oy) * a.Wout + x * a.s_out + ph->ox) * oc + a.co_off
                   : -1L;
    });
}

// ---------------------------------------------------------------- registry
struct WindowEntry {
    int tag, cin, cop, dt, waves;
    void (*fn)(ConvArgs);
};

// (Split FP32 at 192 channels has none: two slices of the window, 86 KB, two stages
// of weights, 72 KB, and the constants are 0.3 KB more than the 160 KB of a CU.)
#define LIC_W(TAG, CIN, MT, NT, NG, WV, ST, DT) {TAG, CIN, MT * 16, DT, WV, gdn_window<TAG, CIN, MT, NT, NG, WV, ST, DT>}
#define LIC_WL(TAG)                                                                          \
    LIC_W(TAG, 128, 8, 4, 2, 4, 4, DT_BF16), LIC_W(TAG, 128, 8, 4, 2, 4, 2, DT_FP8),         \
        LIC_W(TAG, 192, 12, 2, 2, 8, 4, DT_BF16), LIC_W(TAG, 192, 12, 2, 2, 8, 3, DT_FP8),   \
        LIC_W(TAG, 128, 8, 2, 2, 8, 3, DT_F32X)

static const WindowEntry kWindow[] = {LIC_WL(LIC_GS1), LIC_WL(LIC_GS2)};

static const WindowEntry* find_window(int tag, int cin, int cop, int dt)
{
    for (const auto& e : kWindow)
        if (e.tag == tag && e.cin == cin && e.cop == cop && e.dt == dt) return &e;
    return nullptr;
}

bool window_available(int tag, int cin, int cop, int dt) { return find_window(tag, cin, cop, dt) != nullptr; }

hipError_t launch_window(int tag, int cin, int cop, int dt, const ConvArgs& args, hipStream_t stream)
{
    const WindowEntry* e = find_window(tag, cin, cop, dt);
    if (!e) return hipErrorInvalidDeviceFunction;
    const int th = kWindowPixels / args.tw;
    const long tiles = (long)args.n * ((args.Hg + th - 1) / th) * ((args.Wg + args.tw - 1) / args.tw);
    const long nblocks = (tiles + 7) / 8 * 8 * args.nphase;
    hipLaunchKernelGGL(e->fn, dim3((unsigned)nblocks), dim3(64 * e->waves), 0, stream, args);
    return hipGetLastError();
}

}  // namespace lic
