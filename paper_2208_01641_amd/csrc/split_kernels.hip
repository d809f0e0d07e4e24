// Convolution layers of small grids on MFMA (gfx950): split K.  A block owns
// one output tile; KS waves of each of its RG row groups take interleaved K
// chunks and the partial sums are added in LDS in the fixed order 0 .. KS - 1,
// so a result depends on neither timing nor batch.  Covers the hyper layers,
// g_a's last layer, the context model's layers, and the GDN layers of frames
// too small to give every SIMD a wave.
//
// What bounds the direct form (conv_igemm with KSPLIT > 1): every fragment is
// gathered in the MFMA operand layout, 64 lanes on 64 separate 16-byte pieces
// at one piece a clock and CU, which takes longer than the FP32 products; a
// block has one wave per K slot, whose first wave alone adds the partial sums
// and runs the whole epilogue; and the GDN layers give a block all rows of 32
// pixels, which leaves most of the chip without work.  Here
//   * weights come in fragment order, 1 KB contiguous per load, straight into
//     a register ring; pixels in 64-byte runs per quad of lanes into a
//     wave-private LDS ring (no barrier in the K loop), P chunks ahead;
//   * every wave adds the partial sums of its own 16 x 16 tiles and runs the
//     epilogue on them;
//   * GDN blocks take 16 (or 32) pixels with RG groups of 64 rows, and their
//     contraction is spread over all waves, the squares exchanged in LDS.
// FP32 products run on the vector pipe's multipliers: every vector instruction
// between them costs its own 4 clocks and about 10 for the change (measured: 32.2 clocks
// a product alone, 46.5 with one behind each; a bf16 product 16.5, 18.6 with two),
// so the loop has almost none: weights and windows move by scalar
// buffer bases and offsets, and out-of-image taps are a precomputed bit mask
// that sends the lane's offset out of the buffer's range (reads zero).
//
// Chunks, slots, products and the order of all sums are those of conv_igemm:
// the results are the same bits.
//
// Measured against the direct form (kernel time, us): 128 x 128 frame, FP32: g_a's
// second and third layer 70 -> 33, 68 -> 32, g_s's first three 50 -> 23, 36 -> 16,
// 37 -> 17; g_a's third at 360p 73 -> 37, its last at 720p 80 -> 52, at 470 x 834
// 44 -> 31; hyper layers at 720p: h_a 27, 26, 15 -> 22, 14, 10, h_s 13, 19, 40 ->
// 9, 16, 26; e4m3 g_s's second layer at 512 x 768 45 -> 26.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/lic.h"
#include "conv_args.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

// n = beta + gamma (x*x) (1DN: |x|) as in gdn_finish.h, spread over the waves of a
// block: wave w has row block w of every pixel tile (x), and gamma's fragments
// of those rows (G).  The squares' bf16 parts go to LDS as fragments
// [nt][p][part][lane][8]: row block 2p + h fills half h.
template <int TB, int NT, int GP, int EP>
__device__ __forceinline__ void spread_gdn(const ConvArgs& a, const f4 (&x)[NT], const u32x4 (&G)[TB / 2][GP], uint32_t* S, int lane,
                                           int wave, f4 (&y)[NT])
{
    constexpr int NPAIR = TB / 2;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        f4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = a.norm1 ? fabsf(x[nt][i]) : x[nt][i] * x[nt][i];
#pragma unroll
        for (int g = 0; g < GP; ++g) {
            bf16x4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = (__bf16)r[i];
                r[i] -= (float)h[i];
            }
            *reinterpret_cast<bf16x4*>(S + ((nt * NPAIR + (wave >> 1)) * GP + g) * 256 + lane * 4 + (wave & 1) * 2) = h;
        }
    }
    f4 nacc[NT];
    const f4 be = *reinterpret_cast<const f4*>(a.beta + wave * 16 + (lane >> 4) * 4);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) nacc[nt] = be;
    lds_barrier();
#pragma unroll
    for (int p = 0; p < NPAIR; ++p)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            bf16x8 s[GP];
#pragma unroll
            for (int g = 0; g < GP; ++g)
                s[g] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(S + ((nt * NPAIR + p) * GP + g) * 256 + lane * 4));
            auto mul = [&](int g, int h) __attribute__((always_inline)) {
                nacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, G[p][g]), s[h], nacc[nt], 0, 0, 0);
            };
            if constexpr (GP == 3) {
                mul(0, 2);
                mul(1, 1);
                mul(2, 0);
            }
            mul(0, 1);
            mul(1, 0);
            mul(0, 0);
        }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float nv = nacc[nt][i];
            if (EP == EP_GDN)
                y[nt][i] = x[nt][i] * (a.norm1 ? __builtin_amdgcn_rcpf(nv) : __builtin_amdgcn_rsqf(nv));
            else
                y[nt][i] = x[nt][i] * (a.norm1 ? nv : __builtin_amdgcn_sqrtf(nv));
        }
}

// MT x NT: 16-row and 16-pixel tiles per wave; RG: row groups per block (GDN:
// RG MT 16 = all channels); KS: K slots; P: chunks in flight per wave; WPS:
// waves per SIMD the registers are bounded for.
template <int MT, int NT, int RG, int KS, int P, int WPS, int LD, int EP, int DT>
__global__ void __launch_bounds__(64 * RG * KS, WPS) conv_split(ConvArgs a)
{
    using Elem = typename std::conditional<LD == LD_I8, int8_t, typename Prec<DT>::Elem>::type;
    static_assert(DT == DT_F32 || DT == DT_BF16 || DT == DT_FP8, "plain operand forms");
    constexpr bool kGdn = EP == EP_GDN || EP == EP_IGDN;
    constexpr int W = RG * KS;
    constexpr int KCH = Prec<DT>::KCH;
    constexpr int SUB = DT == DT_FP8 ? 2 : 1;
    constexpr int ESZ = (int)sizeof(Elem);
    constexpr int RB = KCH * ESZ;                       // bytes of a pixel and chunk: 16, 32 (symbols), 64, 128
    constexpr int LPR = RB / 16;
    constexpr int PPI = 64 / LPR;                       // pixels per load instruction
    constexpr int NB = (NT * 16 + PPI - 1) / PPI;
    constexpr int BW = NT * 16 * RB / 4 < 256 * NB ? 256 * NB : NT * 16 * RB / 4;   // words per stage
    constexpr int L = NB + MT * SUB;                    // loads per chunk
    constexpr int TB = RG * MT;                         // 16-row blocks of the block's tile
    constexpr int TILES = TB * NT;
    constexpr int GP = DT == DT_F32 ? 3 : 2;            // bf16 parts of gamma and x*x
    constexpr int NPAIR = TB / 2;
    constexpr int kRing = W * P * BW, kRed = KS * TILES * 256, kS = kGdn ? NT * NPAIR * GP * 256 : 0;
    constexpr int kBig = kRing > kRed ? kRing : kRed;
    constexpr int SMW = kBig > kS ? kBig : kS;
    __shared__ __attribute__((aligned(16))) uint32_t smem[SMW];
    __shared__ __attribute__((aligned(16))) float mus[LD == LD_I8 ? 320 : 1];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave % KS, rg = wave / KS;
    const int l16 = lane & 15, kg = lane >> 4;
    const int cin = a.cin;
    int logical = xcd_logical_tile(blockIdx.x, gridDim.x);
    const int cog = logical % a.ncog;
    logical /= a.ncog;
    const int phase = logical % a.nphase;
    const int tile = logical / a.nphase;
    const PhaseDesc* __restrict__ ph = a.ph + phase;
    const int ntaps = ph->ntaps;
    const int tapv = lane < ntaps ? (((int)ph->dy[lane] & 0xffff) | ((int)ph->dx[lane] << 16)) : 0;
    const int HWg = a.Hg * a.Wg;
    const int total = a.n * HWg;
    const int pix0 = tile * (NT * 16);

    // loader: this lane's pixel and 16-byte piece in each of a chunk's loads;
    // a pixel past the end gets an origin no tap brings into the image
    const int lpx = lane / LPR, slot = lane % LPR;
    auto rot = [](int p) { return LPR <= 2 ? 0 : LPR == 4 ? (p >> 1) & 3 : ((p >> 1) & 1) | (((p >> 2) & 1) << 2); };
    // byte offsets count from the first pixel's row (pixels follow each other in
    // memory, so a block's offsets are small whatever the tensor's size); bit t
    // of bad: tap t falls outside the image (or past the last tap)
    const int im0 = pix0 / HWg, y0 = (pix0 - im0 * HWg) / a.Wg;
    const uint8_t* const in0 = static_cast<const uint8_t*>(a.in) + ((long)im0 * a.Hin + y0 * a.s_in) * a.Win * (long)(cin * ESZ);
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
        poff[i] = (uint32_t)((((long)(im - im0) * a.Hin + (y - y0) * a.s_in) * a.Win + ox) * (cin * ESZ)) +
                  (uint32_t)pc[i];
        bad[i] = bad_taps(oy, ox, tapv, ntaps, ph->nx, a.Hin, a.Win);
    }
    // the pixels of this lane's fragments
    int fy[NT], fx[NT], fi[NT];
    bool fv[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int p = pix0 + nt * 16 + l16;
        fv[nt] = p < total;
        const int q = fv[nt] ? p : 0;
        fi[nt] = q / HWg;
        const int r = q - fi[nt] * HWg;
        fy[nt] = r / a.Wg;
        fx[nt] = r - fy[nt] * a.Wg;
    }
    if constexpr (LD == LD_I8) {
        for (int c = threadIdx.x; c < cin; c += 64 * W) mus[c] = a.mu_in[c];
        lds_barrier();
    }

    // this wave's chunks ks, ks + KS, ...: channel slice outer, tap inner
    // (e4m3: the flattened (tap, channel) axis)
    const int K = DT == DT_FP8 ? (ntaps * cin + KCH - 1) / KCH : ntaps * (cin / KCH);
    const int nk = (K - ks + KS - 1) / KS;
    const size_t cstep = (size_t)a.ncog * TB * SUB * 1024;             // bytes of a chunk's weights
    const Buf wbuf = make_buf(static_cast<const uint8_t*>(a.ws) + ph->wtoff * (long)sizeof(typename Prec<DT>::WElem));
    int woff = (int)(ks * cstep) + (cog * TB + rg * MT) * SUB * 1024;
    uint32_t* const ring = smem + wave * (P * BW);
    int i_k = ks, i_t = ks % ntaps, i_s = ks / ntaps;                  // next chunk to load
    const int adv_s = KS / ntaps, adv_t = KS - adv_s * ntaps;
    // lane t: bytes from a window's origin to tap t (no multiplications in the
    // K loop, which would be worth a branch to the compiler)
    const int toffv = ((int)(short)(tapv & 0xffff) * a.Win + (tapv >> 16)) * cin * ESZ;
    auto tap_off = [&](int t) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(toffv, t < ntaps ? t : 0); };
    auto tap = [&](int t, int& dy, int& dx) __attribute__((always_inline)) {
        const int tv = __builtin_amdgcn_readlane(tapv, t < ntaps ? t : 0);
        dy = t < ntaps ? (int)(short)(tv & 0xffff) : -(1 << 20);
        dx = tv >> 16;
    };
    u32x4 A[P][MT][SUB];
    auto issue = [&](uint32_t* st, u32x4 (&Ar)[MT][SUB]) __attribute__((always_inline)) {
        // a chunk's window is the buffer's base moved by its tap; lanes whose
        // tap is out of the image read zero
        if constexpr (DT == DT_FP8) {
            const int f0 = i_k * KCH, tA = f0 / cin, c0 = f0 - tA * cin;
            const int offA = tap_off(tA) + c0, step = tap_off(tA + 1) - cin - tap_off(tA);
            const Buf b = make_buf(in0 + (offA + min(step, 0)));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bool second = c0 + pc[i] >= cin;
                const uint32_t o = (poff[i] + (second ? max(step, 0) : max(-step, 0))) | bit_mask(bad[i], second ? tA + 1 : tA);
                buf_load_lds(b, st + i * 256, o, 0);
            }
        } else {
            const Buf b = make_buf(in0 + (tap_off(i_t) + i_s * (KCH * ESZ)));
#pragma unroll
            for (int i = 0; i < NB; ++i) buf_load_lds(b, st + i * 256, poff[i] | bit_mask(bad[i], i_t), 0);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g = 0; g < SUB; ++g) Ar[mt][g] = buf_load(wbuf, lane * 16 + (mt * SUB + g) * 1024, woff);
        woff += (int)(KS * cstep);
        i_k += KS;
        i_t += adv_t;
        i_s += adv_s;
        if (i_t >= ntaps) {
            i_t -= ntaps;
            ++i_s;
        }
    };

    f4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f4 b = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (DT != DT_FP8) {
            const f4 bl = *reinterpret_cast<const f4*>(a.bias + ((cog * TB + rg * MT + mt) * 16) + kg * 4);
            if (ks == 0) b = bl;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = b;
    }

    // pixel fragments of a chunk as read from its stage; symbols stay raw (with
    // their offsets, which an out-of-image tap must not add) until they are used
    constexpr int KE = KCH / 4;
    struct BRaw {
        u32x4 lo, hi;
    };
    struct I8Raw {
        uint32_t w[2];
        bool ok;
    };
    BRaw Bq[2][NT];
    I8Raw Iq[2][NT];
    float muq[2][LD == LD_I8 ? KE : 1];
    int c_t = ks % ntaps, c_s = ks / ntaps;                            // next chunk to read (symbols)
    const int brow = LPR == 1 ? l16 * 4 + kg : LPR == 2 ? l16 * 8 + kg * 2
                              : l16 * (RB / 4) + (((LPR == 4 ? kg : 2 * kg) ^ rot(l16)) * 4);
    auto readB = [&](const uint32_t* st, int q) __attribute__((always_inline)) {
        if constexpr (LD == LD_I8) {
            int dy, dx;
            tap(c_t, dy, dx);
#pragma unroll
            for (int e = 0; e < KE; e += 4)
                *reinterpret_cast<f4*>(&muq[q][e]) = *reinterpret_cast<const f4*>(mus + c_s * KCH + kg * KE + e);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if constexpr (KE == 4) {
                    Iq[q][nt].w[0] = st[nt * 16 * (RB / 4) + brow];
                } else {
                    const uint2 u = *reinterpret_cast<const uint2*>(st + nt * 16 * (RB / 4) + brow);
                    Iq[q][nt].w[0] = u.x;
                    Iq[q][nt].w[1] = u.y;
                }
                Iq[q][nt].ok = fv[nt] & ((unsigned)(fy[nt] * a.s_in + dy) < (unsigned)a.Hin) &
                               ((unsigned)(fx[nt] * a.s_in + dx) < (unsigned)a.Win);
            }
            c_t += adv_t;
            c_s += adv_s;
            if (c_t >= ntaps) {
                c_t -= ntaps;
                ++c_s;
            }
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                Bq[q][nt].lo = *reinterpret_cast<const u32x4*>(st + nt * 16 * (RB / 4) + brow);
                if constexpr (LPR == 8) Bq[q][nt].hi = *reinterpret_cast<const u32x4*>(st + nt * 16 * (RB / 4) + (brow ^ 4));
            }
        }
    };
    auto multiply = [&](int q, const u32x4 (&Ar)[MT][SUB]) __attribute__((always_inline)) {
        BRaw B[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (LD == LD_I8) {
                float v[KE];
#pragma unroll
                for (int e = 0; e < KE; ++e)
                    v[e] = (float)(int8_t)(Iq[q][nt].w[e / 4] >> (8 * (e % 4))) + (Iq[q][nt].ok ? muq[q][e] : 0.0f);
                if constexpr (DT == DT_F32) {
                    B[nt].lo = __builtin_bit_cast(u32x4, f4{v[0], v[1], v[2], v[3]});
                } else {
                    bf16x8 h;
#pragma unroll
                    for (int e = 0; e < 8; ++e) h[e] = (__bf16)v[e % KE];
                    B[nt].lo = __builtin_bit_cast(u32x4, h);
                }
            } else {
                B[nt] = Bq[q][nt];
                if constexpr (LD == LD_F32_ABS) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) B[nt].lo[e] &= 0x7fffffffu;
                }
            }
        }
        if constexpr (DT == DT_F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = mfma16x16x4(__builtin_bit_cast(f4, Ar[mt][0])[e], __builtin_bit_cast(f4, B[nt].lo)[e], acc[mt][nt]);
        } else if constexpr (DT == DT_BF16) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Ar[mt][0]),
                                                                          __builtin_bit_cast(bf16x8, B[nt].lo), acc[mt][nt], 0, 0, 0);
        } else {
            auto cat = [](const u32x4& lo, const u32x4& hi) {
                return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            };
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        cat(Ar[mt][0], Ar[mt][SUB - 1]), cat(B[nt].lo, B[nt].hi), acc[mt][nt], 0, 0, 0, kE8M0One, 0, kE8M0One);
        }
    };

    // Chunk j sits in stage and register set j % P; once its fragments are in
    // registers and multiplied, the same place takes chunk j + P.  The pixel
    // fragments are read one chunk ahead, in the shadow of the products: the
    // two waves of a SIMD tend to run in step, so a wait between a chunk's
    // read and its products is not filled by the other.  The pixels' loads
    // come before the weights' in each chunk, so waiting for the weights
    // covers both.  (The prologue of the steady loop is unconditional: a load
    // that some path skips makes the compiler wait for everything at the
    // loop's head.)
    static_assert(P % 2 == 0, "fragment sets alternate");
    int k = 0;
    if (nk >= 2 * P) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            issue(ring + j * BW, A[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_vm<(P - 1) * L>();
        readB(ring, 0);
        for (; k + 2 * P <= nk; k += P) {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                wait_vm_lds<(P - 2) * L>();             // chunk j + 1 is in LDS, chunk j's fragments are here
                __builtin_amdgcn_sched_barrier(0);
                readB(ring + (j + 1) % P * BW, (j + 1) & 1);
                multiply(j & 1, A[j]);
                __builtin_amdgcn_sched_barrier(0);
                issue(ring + j * BW, A[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (j < nk) issue(ring + j * BW, A[j]);
        wait_vm<0>();
        if (nk > 0) readB(ring, 0);
    }
    for (; k < nk; k += P) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (k + j >= nk) break;
            wait_vm_lds<0>();
            __builtin_amdgcn_sched_barrier(0);
            if (k + j + 1 < nk) readB(ring + (j + 1) % P * BW, (j + 1) & 1);
            multiply(j & 1, A[j]);
            if (k + j + P < nk) issue(ring + j * BW, A[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // gamma fragments of this wave's rows, loaded before the reduction
    const u32x4* gt = static_cast<const u32x4*>(a.gt);
    u32x4 G[kGdn ? NPAIR : 1][GP];
    if constexpr (kGdn) {
        static_assert(W == TB, "one 16-row block per wave");
#pragma unroll
        for (int p = 0; p < NPAIR; ++p)
#pragma unroll
            for (int g = 0; g < GP; ++g) G[p][g] = gt[((size_t)(p * TB + wave) * GP + g) * 64 + lane];
    }

    // partial sums [slot][row block][nt][lane]; every wave adds its own tiles
    lds_barrier();                                      // the rings have been read
    f4* const red = reinterpret_cast<f4*>(smem);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[((ks * TB + rg * MT + mt) * NT + nt) * 64 + lane] = acc[mt][nt];
    lds_barrier();
    auto summed = [&](int rb, int nt) __attribute__((always_inline)) -> f4 {
        f4 v = red[(rb * NT + nt) * 64 + lane];
#pragma unroll
        for (int s = 1; s < KS; ++s) v += red[((s * TB + rb) * NT + nt) * 64 + lane];
        if constexpr (DT == DT_FP8) {
            // undo the operand scales, then add the bias
            const int c = (cog * TB + rb) * 16 + kg * 4;
            v = v * *reinterpret_cast<const f4*>(a.rscale + c) + *reinterpret_cast<const f4*>(a.bias + c);
        }
        return v;
    };
    const long ldo = a.co_ld ? a.co_ld : a.Co;
    auto out_pix = [&](int nt) __attribute__((always_inline)) -> long {
        return ((long)fi[nt] * a.Hout + fy[nt] * a.s_out + ph->oy) * a.Wout + fx[nt] * a.s_out + ph->ox;
    };
    auto store_act = [&](long idx, const f4& y) __attribute__((always_inline)) {
        if constexpr (DT == DT_F32) {
            *reinterpret_cast<f4*>(static_cast<float*>(a.out) + idx) = y;
        } else if ((DT == DT_FP8 && !a.out_bf16) || (DT == DT_BF16 && a.out_e4m3)) {
            const f4 v = a.out_q * y;
            if (a.sat) {
                const bool s = fabsf(v[0]) > 448.0f || fabsf(v[1]) > 448.0f || fabsf(v[2]) > 448.0f || fabsf(v[3]) > 448.0f;
                const unsigned long long m = __ballot(s);
                if (m && lane == __ffsll((long long)m) - 1) atomicAdd(a.sat, (unsigned long long)__popcll(m));
            }
            *reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(a.out) + idx) = e4m3x2(v[0], v[1]) | (e4m3x2(v[2], v[3]) << 16);
        } else {
            bf16x4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = (__bf16)y[i];
            *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(a.out) + idx) = h;
        }
    };

    if constexpr (kGdn) {
        f4 x[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) x[nt] = summed(wave, nt);
        lds_barrier();                                  // the partial sums have been read
        f4 y[NT];
        spread_gdn<TB, NT, GP, EP>(a, x, G, smem, lane, wave, y);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (fv[nt]) store_act(out_pix(nt) * ldo + a.co_off + wave * 16 + kg * 4, y[nt]);
    } else if constexpr (EP == EP_NONE || EP == EP_RELU) {
#pragma unroll
        for (int t = 0; t < (TILES + W - 1) / W; ++t) {
            const int q = t * W + wave;
            if (TILES % W != 0 && q >= TILES) break;
            const int rb = q / NT;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (nt != q % NT) continue;
                f4 y = summed(rb, nt);
                if constexpr (EP == EP_RELU) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = fmaxf(y[i], 0.0f);
                }
                const int c = (cog * TB + rb) * 16 + kg * 4;
                if (fv[nt] && c < a.Co) store_act(out_pix(nt) * ldo + a.co_off + c, y);
            }
        }
    } else if constexpr (EP == EP_QUANT || EP == EP_INDEX) {
        // the tile's bytes are gathered in LDS and leave as 16-byte pieces,
        // TB of them per pixel (they often go straight to mapped host memory)
        __shared__ __attribute__((aligned(16))) uint32_t obytes[NT * 16][TB * 4];
        __shared__ float ts[64];
        if constexpr (EP == EP_INDEX) {
            if (wave == 0) ts[lane] = lane < 63 ? a.thr[lane] : __builtin_inff();
            lds_barrier();
        }
#pragma unroll
        for (int t = 0; t < (TILES + W - 1) / W; ++t) {
            const int q = t * W + wave;
            if (TILES % W != 0 && q >= TILES) break;
            const int rb = q / NT, c = (cog * TB + rb) * 16 + kg * 4;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (nt != q % NT) continue;
                const f4 y = summed(rb, nt);
                const bool ok = fv[nt] && c < a.Co;
                uint32_t packed = 0;
                if constexpr (EP == EP_QUANT) {
                    const f4 mu = ok ? *reinterpret_cast<const f4*>(a.qmu + c) : f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = fminf(fmaxf(rintf(y[i] - mu[i]), -64.0f), 64.0f);
                        packed |= ((uint32_t)((int)v) & 0xffu) << (8 * i);
                    }
                    if (a.out && ok) *reinterpret_cast<f4*>(static_cast<float*>(a.out) + out_pix(nt) * a.Co + c) = y;
                } else {
                    const float t0 = ts[0];
                    const float inv = a.hs_exp ? 62.0f / (ts[62] - t0) : 62.0f / __log2f(ts[62] / t0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) packed |= (uint32_t)scale_count(y[i], ts, t0, inv, a.hs_exp) << (8 * i);
                    if (a.aux && ok) *reinterpret_cast<f4*>(static_cast<float*>(a.aux) + out_pix(nt) * a.Co + c) = y;
                }
                obytes[nt * 16 + l16][rb * 4 + kg] = packed;
            }
        }
        lds_barrier();
        uint8_t* const dst = static_cast<uint8_t*>(EP == EP_QUANT ? a.aux : a.out);
        for (int q = threadIdx.x; q < NT * 16 * TB; q += 64 * W) {
            const int pl = q / TB, m = q - (q / TB) * TB, p = pix0 + pl;
            if (p < total && (cog * TB + m) * 16 < a.Co) {
                const int im = p / HWg, r = p - im * HWg, y = r / a.Wg, x = r - y * a.Wg;
                const long o = (((long)im * a.Hout + y * a.s_out + ph->oy) * a.Wout + x * a.s_out + ph->ox) * a.Co;
                *reinterpret_cast<u32x4*>(dst + o + (cog * TB + m) * 16) = *reinterpret_cast<const u32x4*>(&obytes[pl][m * 4]);
            }
        }
    } else if constexpr (EP == EP_MSCALE) {
        // rows 2c, 2c + 1 are the mean and the pre-activation scale of latent
        // channel c: lane group kg holds channels c0, c0 + 1
        const int M = a.Co / 2, Wh = a.Wout / 2;
        uint8_t* idxo = static_cast<uint8_t*>(a.out);
        int8_t* symo = static_cast<int8_t*>(a.aux);
        __shared__ float ts[64];
        if (wave == 0) ts[lane] = lane < 63 ? a.thr[lane] : __builtin_inff();
        lds_barrier();
        const float t0 = ts[0];
        const float inv = a.hs_exp ? 62.0f / (ts[62] - t0) : 62.0f / __log2f(ts[62] / t0);
#pragma unroll
        for (int t = 0; t < (TILES + W - 1) / W; ++t) {
            const int q = t * W + wave;
            if (TILES % W != 0 && q >= TILES) break;
            const int rb = q / NT;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (nt != q % NT) continue;
                const f4 v = summed(rb, nt);
                const int c0 = ((cog * TB + rb) * 16 + kg * 4) / 2;
                if (!fv[nt] || c0 >= M) continue;
                // checkerboard-major element: entry fx of the output row
                const long cpix = (((long)fi[nt] * 2 + a.cb_part) * a.Hout + fy[nt] * a.s_out + ph->oy) * Wh + fx[nt];
                const long fpix = out_pix(nt);
                const int e0 = scale_count(v[1], ts, t0, inv, a.hs_exp), e1 = scale_count(v[3], ts, t0, inv, a.hs_exp);
                *reinterpret_cast<uint16_t*>(idxo + cpix * M + c0) = (uint16_t)(e0 | (e1 << 8));
                if (a.ysrc) {
                    const float2 y = *reinterpret_cast<const float2*>(a.ysrc + fpix * M + c0);
                    const float q0 = fminf(fmaxf(rintf(y.x - v[0]), -64.0f), 64.0f);
                    const float q1 = fminf(fmaxf(rintf(y.y - v[2]), -64.0f), 64.0f);
                    if (symo)
                        *reinterpret_cast<uint16_t*>(symo + cpix * M + c0) =
                            (uint16_t)(((uint32_t)((int)q0) & 0xffu) | (((uint32_t)((int)q1) & 0xffu) << 8));
                    *reinterpret_cast<float2*>(a.yq + fpix * M + c0) = make_float2(q0 + v[0], q1 + v[2]);
                } else {
                    *reinterpret_cast<float2*>(a.yq + cpix * M + c0) = make_float2(v[0], v[2]);
                }
            }
        }
    }
}

// The normalisation alone, in place on FP32 activations [pixel][16 TB]: the second
// pass of the smallest GDN layers, whose sums a plain split-K kernel has left
// there.  A block of TB waves takes 16 pixels.  What bounds one small layer is the
// chain of a block's own K loop: with 16 rows a block instead of all, a wave's
// chunk is 4 FP32 products instead of 16, on 8 (12) times the CUs.  128 x 128 frame,
// kernel time of both passes against one (us): g_a's second layer 33 -> 19, its
// third 32 -> 14, g_s's first 27 -> 14.
template <int TB, int EP>
__global__ void __launch_bounds__(64 * TB) gdn_apply(ConvArgs a)
{
    constexpr int GP = 3, NPAIR = TB / 2;
    __shared__ __attribute__((aligned(16))) uint32_t S[NPAIR * GP * 256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int total = a.n * a.Hout * a.Wout, p = blockIdx.x * 16 + (lane & 15);
    float* const px = static_cast<float*>(a.out) + (long)(p < total ? p : 0) * (16 * TB) + wave * 16 + (lane >> 4) * 4;
    const u32x4* gt = static_cast<const u32x4*>(a.gt);
    f4 x[1], y[1];
    x[0] = *reinterpret_cast<const f4*>(px);
    u32x4 G[NPAIR][GP];
#pragma unroll
    for (int q = 0; q < NPAIR; ++q)
#pragma unroll
        for (int g = 0; g < GP; ++g) G[q][g] = gt[((size_t)(q * TB + wave) * GP + g) * 64 + lane];
    spread_gdn<TB, 1, GP, EP>(a, x, G, S, lane, wave, y);
    if (p < total) *reinterpret_cast<f4*>(px) = y[0];
}

hipError_t launch_gdn_apply(int cop, int ep, const ConvArgs& a, hipStream_t stream)
{
    const dim3 grid((unsigned)(((long)a.n * a.Hout * a.Wout + 15) / 16));
    if (cop == 128)
        hipLaunchKernelGGL((ep == EP_GDN ? gdn_apply<8, EP_GDN> : gdn_apply<8, EP_IGDN>), grid, dim3(512), 0, stream, a);
    else
        hipLaunchKernelGGL((ep == EP_GDN ? gdn_apply<12, EP_GDN> : gdn_apply<12, EP_IGDN>), grid, dim3(768), 0, stream, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- registry
struct SplitEntry {
    SplitKey key;
    void (*fn)(ConvArgs);
};

#define LIC_S(MT, NT, RG, KS, P, WPS, LD, EP, DT) \
    {{MT, NT, RG, KS, LD, EP, DT}, conv_split<MT, NT, RG, KS, P, WPS, LD, EP, DT>}
// Eight slots: 64-row tiles of 32 and 16 pixels, 32- and 16-row tiles of 16 pixels.
// Four slots, which take at least 512 tiles of 64 x 32 an image: 64-row tiles, in
// the reduced forms of 32 pixels.
#define LIC_SE(LD, EP, DT)                                                                                    \
    LIC_S(4, 2, 1, 8, 2, 4, LD, EP, DT), LIC_S(4, 1, 1, 8, 4, 4, LD, EP, DT), LIC_S(2, 1, 1, 8, 4, 6, LD, EP, DT), \
        LIC_S(1, 1, 1, 8, 4, 8, LD, EP, DT), LIC_S(4, 2, 1, 4, 2, 4, LD, EP, DT)
#define LIC_SE4(LD, EP, DT) LIC_SE(LD, EP, DT), LIC_S(4, 1, 1, 4, 4, 4, LD, EP, DT)
// (e4m3 fragments are twice as large)
#define LIC_SEF(LD, EP, DT)                                                                                   \
    LIC_S(4, 2, 1, 8, 2, 2, LD, EP, DT), LIC_S(4, 1, 1, 8, 2, 2, LD, EP, DT), LIC_S(2, 1, 1, 8, 2, 2, LD, EP, DT), \
        LIC_S(1, 1, 1, 8, 4, 4, LD, EP, DT), LIC_S(4, 2, 1, 4, 2, 2, LD, EP, DT)
// GDN layers: 128 and 192 rows; 32-pixel tiles in FP32 only (the reduced forms
// leave for the staged kernel before)
#define LIC_SG(LD, EP)                                                                                        \
    LIC_S(4, 1, 2, 4, 4, 4, LD, EP, DT_F32), LIC_S(4, 2, 2, 4, 4, 2, LD, EP, DT_F32),                          \
        LIC_S(4, 1, 3, 4, 4, 3, LD, EP, DT_F32), LIC_S(4, 2, 3, 4, 2, 3, LD, EP, DT_F32)
#define LIC_SGB(LD, EP) LIC_S(4, 1, 2, 4, 4, 4, LD, EP, DT_BF16), LIC_S(4, 1, 3, 4, 4, 3, LD, EP, DT_BF16)
#define LIC_SGF(LD, EP) LIC_S(4, 1, 2, 4, 2, 2, LD, EP, DT_FP8), LIC_S(4, 1, 3, 4, 2, 3, LD, EP, DT_FP8)

// the sums of the smallest GDN layers (a second pass normalises)
#define LIC_SS(LD) LIC_S(1, 1, 1, 4, 8, 4, LD, EP_NONE, DT_F32)

static const SplitEntry kSplit[] = {
    LIC_SS(LD_F32), LIC_S(2, 1, 1, 4, 4, 6, LD_F32, EP_NONE, DT_F32),
    LIC_SS(LD_I8), LIC_S(2, 1, 1, 4, 4, 4, LD_I8, EP_NONE, DT_F32),
    LIC_SE4(LD_F32, EP_RELU, DT_F32),  LIC_SE4(LD_F32_ABS, EP_RELU, DT_F32), LIC_SE4(LD_I8, EP_RELU, DT_F32),
    LIC_SE4(LD_F32, EP_QUANT, DT_F32), LIC_SE(LD_F32, EP_QUANT, DT_BF16),    LIC_SEF(LD_F32, EP_QUANT, DT_FP8),
    LIC_SE4(LD_F32, EP_INDEX, DT_F32), LIC_SE4(LD_F32, EP_NONE, DT_F32),     LIC_SE4(LD_F32, EP_MSCALE, DT_F32),
    LIC_SG(LD_F32, EP_GDN),  LIC_SG(LD_F32, EP_IGDN),  LIC_SG(LD_I8, EP_IGDN),
    LIC_SGB(LD_F32, EP_GDN), LIC_SGB(LD_F32, EP_IGDN), LIC_SGB(LD_I8, EP_IGDN),
    LIC_SGF(LD_F32, EP_GDN), LIC_SGF(LD_F32, EP_IGDN),
};

bool split_available(const SplitKey& k)
{
    for (const auto& e : kSplit)
        if (e.key == k) return true;
    return false;
}

hipError_t launch_split(const SplitKey& k, const ConvArgs& args, int nblocks, hipStream_t stream)
{
    for (const auto& e : kSplit)
        if (e.key == k) {
            hipLaunchKernelGGL(e.fn, dim3(nblocks), dim3(64 * k.rg * k.ks), 0, stream, args);
            return hipGetLastError();
        }
    return hipErrorInvalidDeviceFunction;
}

}  // namespace lic
