// GDN / IGDN convolution layers of whole frames on MFMA (gfx950): the
// implicit GEMM of conv_kernels.hip with both operands staged in LDS.
//
// What bounds the direct form: the MFMA operand layout puts 16 pixels in 16
// neighbouring lanes, so a gather straight into registers sends 64 lanes to
// 64 separate 16-byte pieces, and the vector memory path takes one piece a
// clock (measured 16.0 bytes a clock and CU, against 62.6 when the four lanes
// of a quad read one 64-byte run).  Here every global load is such a run:
//   * weights are packed in fragment order (lane by lane, 1 KB per fragment),
//     so a chunk's weight tile goes from memory to LDS linearly and is read
//     back linearly (LDS reads at 235 bytes a clock; 64-byte rows padded to 80
//     bytes gave 125);
//   * a wave loads its pixels' channel runs with consecutive lanes on one
//     pixel; the 16-byte pieces of a row are stored rotated by the pixel
//     index (an exclusive or), which makes the fragment reads conflict-free
//     (a b128 read takes lanes 0-7 with 16-23, 8-15 with 24-31, ... together);
//   * gamma comes in fragment order too, and the outputs are transposed in LDS
//     so that each pixel's channels leave in whole 16-byte pieces.
// All of it goes straight from memory to LDS (buffer loads with the lds bit)
// into a ring of ST stages, ST - 1 chunks ahead, with one barrier per chunk and a
// wait that leaves the later chunks in flight.  Grids that give a SIMD one
// wave have nothing to hide a chunk's LDS reads and the splitting of its
// pixels behind: where a third stage fits, those are done for the next chunk among
// the products of this one (720p split-FP32 GA2 95 -> 87 us, GS0 59 -> 50; 360p GA1
// 95 -> 87).
//
// The products, their order and the order of the channels and taps are those
// of conv_igemm, so the results are the same bits; with KS = 4 those of the
// split-K kernels, whose four sums a wave then keeps in its own registers.
//
// Measured against the direct form (kernel time, us): 720p split-FP32 GA1
// 289 -> 252, GS2 382 -> 333; bf16 GA1 89 -> 68, GS2 129 -> 104; e4m3 GA1 50 ->
// 40, GS2 90 -> 72; four 1080p frames at 192 channels bf16 GA1 1838 -> 1005,
// GS2 2780 -> 1428, e4m3 GA1 1041 -> 608, GS2 1917 -> 988.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/lic.h"
#include "conv_args.h"
#include "gdn_finish.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

// WAVES: 4 with two blocks per CU, or 8 with one where two blocks' stages do
// not fit its 160 KB of LDS (either way two waves per SIMD, 256 registers).
template <int TAG, int CIN, int MT, int NT, int WAVES, int ST, int KS, int LD, int EP, int DT>
__global__ void __launch_bounds__(64 * WAVES, WAVES == 4 ? 2 : 1) gdn_staged(ConvArgs a)
{
    using Elem = typename std::conditional<LD == LD_I8, int8_t, typename Prec<DT>::Elem>::type;
    static_assert(DT == DT_F32X || DT == DT_BF16 || DT == DT_FP8, "matrix-core forms");
    static_assert(LD == LD_F32 || (LD == LD_I8 && DT != DT_FP8), "NHWC activations or symbols");
    constexpr int KCH = Prec<DT>::KCH;
    constexpr int SUB = DT == DT_F32X ? 3 : DT == DT_FP8 ? 2 : 1;  // 1 KB weight fragments per 16 rows and chunk
    constexpr int ESZ = (int)sizeof(Elem);
    constexpr int RB = KCH * ESZ;                                  // bytes of a pixel and chunk
    constexpr int LPR = RB / 16;                                   // lanes (16-byte pieces) per pixel
    constexpr int PPI = 64 / LPR;                                  // pixels per load instruction
    constexpr int NB = (NT * 16 + PPI - 1) / PPI;                  // pixel loads per wave and chunk
    constexpr int AP = MT * SUB;                                   // weight fragments (KB) per chunk
    constexpr int AW = (AP + WAVES - 1) / WAVES;                   // loads of them per wave (past the end: the last again)
    // stages of weights (ST) and of pixels: three of pixels where three of both do
    // not fit (not e4m3, which has nothing to convert: 40.1 us so, 41.4 with it)
    constexpr int PS = ST == 2 && DT == DT_F32X && NT == 1 ? 3 : ST;
    static_assert(RB == 32 || RB == 64 || RB == 128, "whole pieces per pixel");
    constexpr int STW = AP * 256, PSW = WAVES * NB * 256;           // words per stage
    constexpr int RINGW = ST * STW + PS * PSW;
    constexpr int MUW = LD == LD_I8 ? CIN : 0;                     // the symbols' offsets, behind the stages
    constexpr int OUTW = gdn_out_words(MT, WAVES, DT);
    constexpr int SMW = RINGW + MUW > OUTW ? RINGW + MUW : OUTW;
    static_assert(SMW * 4 <= (WAVES == 4 ? 81920 : 163840), "two waves per SIMD");
    __shared__ __attribute__((aligned(16))) uint32_t smem[SMW];
    uint32_t* const pring = smem + ST * STW;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    int logical = xcd_logical_tile(blockIdx.x, gridDim.x);
    const int phase = logical % a.nphase;
    const int tile = logical / a.nphase;
    const PhaseDesc* __restrict__ ph = a.ph + phase;
    const int ntaps = ph->ntaps;
    // lane t keeps the offsets of tap t
    const int tapv = lane < ntaps ? (((int)ph->dy[lane] & 0xffff) | ((int)ph->dx[lane] << 16)) : 0;
    const Buf wbuf = make_buf(static_cast<const uint8_t*>(a.wt) + ph->wtoff * (DT == DT_F32X ? 6 : (int)sizeof(typename Prec<DT>::WElem)));
    const int HWg = a.Hg * a.Wg;
    const int total = a.n * HWg;
    const int pix0 = (tile * WAVES + wave) * (NT * 16);

    // loader: this lane's pixel and piece in each of the NB loads of a chunk.
    // A pixel past the end gets an origin no tap brings into the image.
    const int lpx = lane / LPR, slot = lane % LPR;
    auto rot = [](int p) { return LPR == 2 ? 0 : LPR == 4 ? (p >> 1) & 3 : ((p >> 1) & 1) | (((p >> 2) & 1) << 2); };
    // byte offsets count from the wave's first pixel's row (pixels follow each
    // other in memory, so they are small whatever the tensor's size); bit t of
    // bad: tap t falls outside the image (or past the last tap)
    const int im0 = pix0 / HWg, y0 = (pix0 - im0 * HWg) / a.Wg;
    const uint8_t* const in0 = static_cast<const uint8_t*>(a.in) + ((long)im0 * a.Hin + y0 * a.s_in) * a.Win * (long)(CIN * ESZ);
    int pc[NB];
    uint32_t poff[NB], bad[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int pl = i * PPI + lpx;
        const int p = pl < NT * 16 ? pix0 + pl : total;
        const int q = p < total ? p : pix0;
        const int im = q / HWg, r = q - im * HWg;
        const int y = r / a.Wg, x = r - y * a.Wg;
        const int oy = p < total ? y * a.s_in : -(1 << 20), ox = x * a.s_in;
        pc[i] = (slot ^ rot(pl & 15)) * 16;
        poff[i] = (uint32_t)((((long)(im - im0) * a.Hin + (y - y0) * a.s_in) * a.Win + ox) * (CIN * ESZ)) +
                  (uint32_t)pc[i];
        bad[i] = bad_taps(oy, ox, tapv, ntaps, ph->nx, a.Hin, a.Win);
    }

    constexpr int KC = DT == DT_FP8 ? 1 : CIN / KCH;
    const int nk = DT == DT_FP8 ? (ntaps * CIN + KCH - 1) / KCH : ntaps * KC;
    int i_t = 0, i_s = 0, i_k = 0, i_st = 0, w_k = 0, w_st = 0;    // next chunk to load: tap, channel slice, index, stage; weights
    const int toffv = ((int)(short)(tapv & 0xffff) * a.Win + (tapv >> 16)) * (CIN * ESZ);   // bytes to tap t
    auto tap_off = [&](int t) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(toffv, t < ntaps ? t : 0); };
    auto tap = [&](int t, int& dy, int& dx) __attribute__((always_inline)) {
        const int tv = __builtin_amdgcn_readlane(tapv, t < ntaps ? t : 0);
        dy = t < ntaps ? (int)(short)(tv & 0xffff) : -(1 << 20);
        dx = tv >> 16;
    };
    auto issue_w = [&]() __attribute__((always_inline)) {
        uint32_t* const st = smem + w_st * STW;
#pragma unroll
        for (int u = 0; u < AW; ++u) {
            const int f = AP % WAVES == 0 ? wave * AW + u : min(wave * AW + u, AP - 1);
            buf_load_lds(wbuf, st + f * 256, lane * 16, (w_k * AP + f) * 1024);
        }
        ++w_k;
        if (++w_st == ST) w_st = 0;
    };
    auto issue_p = [&]() __attribute__((always_inline)) {
        // a chunk's window is the buffer's base moved by its tap; lanes whose
        // tap is out of the image read zero
        uint32_t* const sb = pring + i_st * PSW + wave * NB * 256;
        if constexpr (DT == DT_FP8) {
            const int f0 = i_k * KCH, tA = f0 / CIN, c0 = f0 - tA * CIN;
            const int step = CIN % KCH != 0 ? tap_off(tA + 1) - CIN - tap_off(tA) : 0;
            const Buf b = make_buf(in0 + (tap_off(tA) + c0 + min(step, 0)));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bool second = CIN % KCH != 0 && c0 + pc[i] >= CIN;
                buf_load_lds(b, sb + i * 256, (poff[i] + (second ? max(step, 0) : max(-step, 0))) | bit_mask(bad[i], second ? tA + 1 : tA), 0);
            }
        } else {
            const Buf b = make_buf(in0 + (tap_off(i_t) + i_s * (KCH * ESZ)));
#pragma unroll
            for (int i = 0; i < NB; ++i) buf_load_lds(b, sb + i * 256, poff[i] | bit_mask(bad[i], i_t), 0);
        }
        if (++i_t == ntaps) {
            i_t = 0;
            ++i_s;
        }
        ++i_k;
        if (++i_st == PS) i_st = 0;
    };

    // symbols: the offsets in LDS, and the pixels of this lane's fragments
    // (an out-of-image tap reads symbol 0 and must not add the offset)
    float* const mus = reinterpret_cast<float*>(smem + RINGW);
    int fy[NT], fx[NT], r_t = 0, r_s = 0;
    if constexpr (LD == LD_I8) {
        for (int c = threadIdx.x; c < CIN; c += 64 * WAVES) mus[c] = a.mu_in[c];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int p = pix0 + nt * 16 + l16;
            const int q = p < total ? p : 0;
            const int r = q - (q / HWg) * HWg;
            fy[nt] = p < total ? (r / a.Wg) * a.s_in : -(1 << 20);
            fx[nt] = (r - (r / a.Wg) * a.Wg) * a.s_in;
        }
    }

    // KS sums per output, chunk k to sum k % KS (the K slots of a split layer)
    f4 part[KS][MT][NT];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            f4 b = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (DT != DT_FP8)
                if (s == 0) b = *reinterpret_cast<const f4*>(a.bias + mt * 16 + kg * 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) part[s][mt][nt] = b;
        }

    // With a third stage the next chunk's fragments are read (and the pixels'
    // split or converted) in the shadow of this one's products, before its
    // barrier; else they are read first and the loads of a later chunk are
    // issued in their shadow.
    constexpr bool BAHEAD = PS >= 3, AAHEAD = ST >= 3;
    constexpr int PF = DT == DT_F32X ? 2 : 4;                      // weight fragments held
    static_assert(MT % PF == 0, "fragment slots");
    const int brow = LPR == 2 ? l16 * 8 + kg * 2 : l16 * (RB / 4) + (((LPR == 4 ? kg : 2 * kg) ^ rot(l16)) * 4);
    struct Pix {                                                   // a pixel fragment as the products take it
        u32x4 p[DT == DT_BF16 ? 1 : DT == DT_FP8 ? 2 : 3];
    };
    u32x4 Bl[NT], Bh[NT], A[PF][SUB];
    uint2 Bs[NT];
    f4 mu[2];
    bool ok[NT];
    Pix N[NT];
    int ra_st = 0, rb_st = 0;
    auto readA = [&](int mt) __attribute__((always_inline)) {
        const uint32_t* const as = smem + ra_st * STW + lane * 4;
#pragma unroll
        for (int g = 0; g < SUB; ++g) A[mt % PF][g] = *reinterpret_cast<const u32x4*>(as + (mt * SUB + g) * 256);
    };
    auto readB = [&]() __attribute__((always_inline)) {
        const uint32_t* const bs = pring + rb_st * PSW + wave * NB * 256;
        if constexpr (LD == LD_I8) {
            int dy, dx;
            tap(r_t, dy, dx);
            const int c = r_s < KC ? r_s * KCH : 0;
#pragma unroll
            for (int e = 0; e < 2; ++e) mu[e] = *reinterpret_cast<const f4*>(mus + c + kg * 8 + e * 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                Bs[nt] = *reinterpret_cast<const uint2*>(bs + brow + nt * 16 * (RB / 4));
                ok[nt] = ((unsigned)(fy[nt] + dy) < (unsigned)a.Hin) & ((unsigned)(fx[nt] + dx) < (unsigned)a.Win);
            }
            if (++r_t == ntaps) {
                r_t = 0;
                ++r_s;
            }
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                Bl[nt] = *reinterpret_cast<const u32x4*>(bs + brow + nt * 16 * (RB / 4));
                if constexpr (LPR == 8) Bh[nt] = *reinterpret_cast<const u32x4*>(bs + (brow ^ 4) + nt * 16 * (RB / 4));
            }
        }
        if (++rb_st == PS) rb_st = 0;
    };
    auto prepare = [&](int nt) __attribute__((always_inline)) -> Pix {
        Pix r;
        if constexpr (LD == LD_F32 && DT != DT_F32X) {
            r.p[0] = Bl[nt];
            if constexpr (DT == DT_FP8) r.p[1] = Bh[nt];
        } else {
            float v[8];
            if constexpr (LD == LD_I8) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = (float)(int8_t)((e < 4 ? Bs[nt].x : Bs[nt].y) >> (8 * (e % 4))) + (ok[nt] ? mu[e / 4][e % 4] : 0.0f);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = __builtin_bit_cast(f4, e < 4 ? Bl[nt] : Bh[nt])[e % 4];
            }
            if constexpr (DT == DT_F32X) {
                const Split3 x = split3(v);
#pragma unroll
                for (int g = 0; g < 3; ++g) r.p[g] = __builtin_bit_cast(u32x4, x.p[g]);
            } else {
                bf16x8 h;
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = (__bf16)v[e];
                r.p[0] = __builtin_bit_cast(u32x4, h);
            }
        }
        return r;
    };
    auto step = [&](f4 (&acc)[MT][NT], auto more) __attribute__((always_inline)) {
        if constexpr (!BAHEAD) readB();
        if constexpr (!AAHEAD) {
#pragma unroll
            for (int mt = 0; mt < PF; ++mt) readA(mt);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            issue_w();
            issue_p();
        }
        Pix C[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) C[nt] = BAHEAD ? N[nt] : prepare(nt);
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
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[pa[s]]),
                                                                              __builtin_bit_cast(bf16x8, C[nt].p[pbx[s]]), acc[mt][nt], 0, 0, 0);
            } else if constexpr (DT == DT_BF16) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[0]),
                                                                          __builtin_bit_cast(bf16x8, C[nt].p[0]), acc[mt][nt], 0, 0, 0);
            } else {
                auto cat = [](const u32x4& lo, const u32x4& hi) {
                    return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
                };
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        cat(W[0], W[SUB - 1]), cat(C[nt].p[0], C[nt].p[1]), acc[mt][nt], 0, 0, 0, kE8M0One, 0, kE8M0One);
            }
            // the fragments of the rows to come; before the last PF rows, the next chunk's
            if (mt + PF == MT) {
                if (++ra_st == ST) ra_st = 0;
            }
            if (mt + PF < MT || AAHEAD) readA((mt + PF) % MT);
            if (BAHEAD && mt + PF == MT - 1) readB();
            if (BAHEAD && mt + NT >= MT) N[mt + NT - MT] = prepare(mt + NT - MT);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Step k issues weights k + ST - 1 and pixels k + PS - 1 into the stages of
    // chunk k - 1; it needs chunk k, or k + 1 of what is read ahead, and waits
    // with the loads behind those in flight.
    constexpr int LATER = ST == PS ? (AAHEAD ? ST - 3 : ST - 2) * (AW + NB) : 0;
    static_assert(ST == PS || (ST == 2 && PS == 3), "the last step's loads are needed");
#pragma unroll
    for (int j = 0; j < PS - 1; ++j) {
        if (j < ST - 1 && j < nk) issue_w();
        if (j < nk) issue_p();
    }
    wait_vm<0>();                                       // (the compiler then adds no waits of its own to the loop)
    lds_barrier();
    if constexpr (BAHEAD) {
        readB();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) N[nt] = prepare(nt);
    }
    if constexpr (AAHEAD) {
#pragma unroll
        for (int mt = 0; mt < PF; ++mt) readA(mt);
    }
    if constexpr (KS == 1) {
        int k = 0;
        for (; k + PS - 1 < nk; ++k) {
            wait_vm<LATER>();
            lds_barrier();
            step(part[0], std::true_type{});
        }
        for (; k < nk; ++k) {
            wait_vm<0>();
            lds_barrier();
            if (ST < PS && k + ST - 1 < nk) issue_w();
            step(part[0], std::false_type{});
        }
    } else {
        static_assert(ST == PS, "one condition for both rings");
#pragma unroll 1
        for (int k = 0; k < nk; k += KS)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (k + s >= nk) break;
                if (k + s + ST - 2 < nk) wait_vm<LATER>();
                else wait_vm<0>();
                lds_barrier();
                step(part[s], k + s + ST - 1 < nk);
                // (else the compiler moves the products behind the loop's exits)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(part[s][mt][nt]));
            }
    }
    f4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            acc[mt][nt] = part[0][mt][nt];
#pragma unroll
            for (int s = 1; s < KS; ++s) acc[mt][nt] += part[s][mt][nt];
        }
    lds_barrier();                                      // every stage is free

    const long oc = a.co_ld ? a.co_ld : a.Co;
    gdn_finish<MT, NT, NT, WAVES, SMW, EP, DT, false>(a, nullptr, acc, smem, lane, wave, [&](int nt) __attribute__((always_inline)) {
        const int p = pix0 + nt * 16 + l16;
        const int q = p < total ? p : 0;
        const int im = q / HWg, r = q - im * HWg;
        const int y = r / a.Wg, x = r - y * a.Wg;
        return p < total ? (((long)im * a.Hout + y * a.s_out + ph->oy) * a.Wout + x * a.s_out + ph->ox) * oc + a.co_off : -1L;
    });
}

// ---------------------------------------------------------------- registry
struct GdnEntry {
    KernelKey key;
    void (*fn)(ConvArgs);
};

#define LIC_G(TAG, CIN, MT, NT, WV, ST, LD, EP, DT) \
    {{TAG, CIN, MT, NT, WV, 1, LD, EP, DT}, gdn_staged<TAG, CIN, MT, NT, WV, ST, 1, LD, EP, DT>}
// four K slots (layers whose grid of one image would leave SIMDs idle)
#define LIC_G4(TAG, CIN, MT, ST, LD, EP, DT) {{TAG, CIN, MT, 1, 4, 4, LD, EP, DT}, gdn_staged<TAG, CIN, MT, 1, 4, ST, 4, LD, EP, DT>}
#define LIC_GK(TAG, EP)                                                                                        \
    LIC_G4(TAG, 128, 8, 4, LD_F32, EP, DT_BF16), LIC_G4(TAG, 192, 12, 4, LD_F32, EP, DT_BF16),                 \
        LIC_G4(TAG, 128, 8, 3, LD_F32, EP, DT_FP8), LIC_G4(TAG, 192, 12, 2, LD_F32, EP, DT_FP8)
// one layer at 128 and 192 channels; NT = 1 for grids that would leave SIMDs
// idle with two 16-pixel tiles per wave (its stages are smaller: more of them)
#define LIC_GX(TAG, EP)                                                                                        \
    LIC_G(TAG, 128, 8, 2, 4, 2, LD_F32, EP, DT_F32X), LIC_G(TAG, 128, 8, 1, 4, 2, LD_F32, EP, DT_F32X),        \
        LIC_G(TAG, 192, 12, 1, 8, 2, LD_F32, EP, DT_F32X)
#define LIC_GB(TAG, EP)                                                                                        \
    LIC_G(TAG, 128, 8, 2, 4, 4, LD_F32, EP, DT_BF16), LIC_G(TAG, 128, 8, 1, 4, 4, LD_F32, EP, DT_BF16),        \
        LIC_G(TAG, 192, 12, 2, 4, 3, LD_F32, EP, DT_BF16), LIC_G(TAG, 192, 12, 1, 4, 4, LD_F32, EP, DT_BF16)
// (e4m3 at 128 channels: unsplit K comes with two tiles a wave, but for GA2)
#define LIC_GF(TAG, EP)                                                                                        \
    LIC_G(TAG, 128, 8, 2, 4, 2, LD_F32, EP, DT_FP8), LIC_G(TAG, 192, 12, 2, 4, 2, LD_F32, EP, DT_FP8), LIC_G(TAG, 192, 12, 1, 4, 2, LD_F32, EP, DT_FP8)

static const GdnEntry kGdn[] = {
    LIC_GX(LIC_GA1, EP_GDN), LIC_GX(LIC_GA2, EP_GDN), LIC_GX(LIC_GS1, EP_IGDN), LIC_GX(LIC_GS2, EP_IGDN),
    LIC_GB(LIC_GA1, EP_GDN), LIC_GB(LIC_GA2, EP_GDN), LIC_GB(LIC_GS1, EP_IGDN), LIC_GB(LIC_GS2, EP_IGDN),
    LIC_GF(LIC_GA1, EP_GDN), LIC_GF(LIC_GA2, EP_GDN), LIC_G(LIC_GA2, 128, 8, 1, 4, 3, LD_F32, EP_GDN, DT_FP8),
    LIC_GF(LIC_GS1, EP_IGDN), LIC_GF(LIC_GS2, EP_IGDN),
    LIC_GK(LIC_GA1, EP_GDN), LIC_GK(LIC_GA2, EP_GDN), LIC_GK(LIC_GS1, EP_IGDN), LIC_GK(LIC_GS2, EP_IGDN),
    LIC_G4(LIC_GS0, 192, 8, 4, LD_I8, EP_IGDN, DT_BF16), LIC_G4(LIC_GS0, 192, 8, 4, LD_F32, EP_IGDN, DT_BF16),
    LIC_G4(LIC_GS0, 320, 12, 4, LD_I8, EP_IGDN, DT_BF16),
    // g_s from symbols, and from y_hat (context model)
    LIC_G(LIC_GS0, 192, 8, 2, 4, 2, LD_I8, EP_IGDN, DT_F32X), LIC_G(LIC_GS0, 192, 8, 1, 4, 2, LD_I8, EP_IGDN, DT_F32X),
    LIC_G(LIC_GS0, 192, 8, 2, 4, 4, LD_I8, EP_IGDN, DT_BF16), LIC_G(LIC_GS0, 192, 8, 1, 4, 4, LD_I8, EP_IGDN, DT_BF16),
    LIC_G(LIC_GS0, 192, 8, 2, 4, 2, LD_F32, EP_IGDN, DT_F32X), LIC_G(LIC_GS0, 192, 8, 1, 4, 2, LD_F32, EP_IGDN, DT_F32X),
    LIC_G(LIC_GS0, 192, 8, 2, 4, 4, LD_F32, EP_IGDN, DT_BF16), LIC_G(LIC_GS0, 192, 8, 1, 4, 4, LD_F32, EP_IGDN, DT_BF16),
    LIC_G(LIC_GS0, 320, 12, 1, 8, 2, LD_I8, EP_IGDN, DT_F32X), LIC_G(LIC_GS0, 320, 12, 1, 4, 4, LD_I8, EP_IGDN, DT_BF16),
};

bool gdn_available(const KernelKey& k)
{
    for (const auto& e : kGdn)
        if (e.key == k) return true;
    return false;
}

hipError_t launch_gdn(const KernelKey& k, const ConvArgs& args, int nblocks, hipStream_t stream)
{
    for (const auto& e : kGdn)
        if (e.key == k) {
            hipLaunchKernelGGL(e.fn, dim3(nblocks), dim3(64 * k.waves), 0, stream, args);
            return hipGetLastError();
        }
    return hipErrorInvalidDeviceFunction;
}

}  // namespace lic
