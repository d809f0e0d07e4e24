// GDN contraction and output stores of the kernels whose waves hold every
// channel of their pixels (gdn_kernels.hip, window_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "conv_args.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

// words of LDS that the stores of WAVES waves need (16 pixels each; a row is
// padded by 16 bytes, which spreads the rows over the banks)
constexpr int gdn_out_words(int MT, int WAVES, int DT)
{
    return WAVES * 16 * (DT == DT_F32X ? MT * 16 + 4 : MT * 8 + 4);
}

// n = beta + gamma (x*x) as in conv_igemm: x*x and gamma in GP bf16 parts, 32
// channels per K chunk; gamma slice p = [mt][part][lane][8].  acc: MT x NT tiles
// of 16 channels x 16 pixels before the scales (e4m3) and the normalisation;
// smem (SMW words): free for every wave.  The contraction takes NG pixel tiles
// at a time (fewer registers where all of gamma fits LDS).  dest(nt) = the
// lane's pixel (lane % 16 of tile nt) as an output element offset, or -1.
// CST: bias, beta and (e4m3) scales are in LDS at cst.
template <int MT, int NT, int NG, int WAVES, int SMW, int EP, int DT, bool CST, class Dest>
__device__ __forceinline__ void gdn_finish(const ConvArgs& a, const float* cst, f4 (&acc)[MT][NT], uint32_t* smem, int lane, int wave,
                                           const Dest& dest)
{
    constexpr int GP = DT == DT_F32X ? 3 : 2;           // bf16 parts of gamma and x*x
    constexpr int NPAIR = MT / 2;
    constexpr int GSW = MT * GP * 256;                  // words per 32-channel gamma slice
    constexpr int GSL = SMW / GSW < NPAIR ? SMW / GSW : NPAIR;   // slices in LDS at once
    static_assert(GSL >= 2, "gamma ring");
    static_assert(NG == NT || (NT % NG == 0 && GSL == NPAIR), "all of gamma stays for the later pixel tiles");
    static_assert(SMW >= gdn_out_words(MT, WAVES, DT), "room for the stores");
    constexpr int GW = (MT * GP + WAVES - 1) / WAVES;   // loads of a slice per wave
    constexpr int CO = MT * 16;
    const int l16 = lane & 15, kg = lane >> 4;
    const Buf gbuf = make_buf(a.gt);
    auto g_issue = [&](int p) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < GW; ++u) {
            const int f = MT * GP % WAVES == 0 ? wave * GW + u : min(wave * GW + u, MT * GP - 1);
            buf_load_lds(gbuf, smem + (p % GSL) * GSW + f * 256, lane * 16, (p * (MT * GP) + f) * 1024);
        }
    };
    if constexpr (DT == DT_FP8) {
        // undo the operand scales, then add the bias
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f4 rs = *reinterpret_cast<const f4*>((CST ? cst + 2 * CO : a.rscale) + mt * 16 + kg * 4);
            const f4 b = *reinterpret_cast<const f4*>((CST ? cst : a.bias) + mt * 16 + kg * 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = acc[mt][nt] * rs + b;
            if (mt % 2 == 1) __builtin_amdgcn_sched_barrier(0);      // few scales in registers at a time
        }
    }
    // slices issued so far, before pair p (ring: one more per pair from pair 1 on)
    constexpr bool RES = GSL == NPAIR;
    constexpr int HALF = (NPAIR + 1) / 2;
#pragma unroll
    for (int p = 0; p < GSL; ++p) g_issue(p);
    // what the registers left by the sums hold: gamma fragments read ahead of
    // their use, and the next pair's squares
    constexpr bool TIGHT = MT * (NT + NG) > 32;
    constexpr int PG = MT == 8 && (!TIGHT || GP == 2) ? 4 : 2, NSQ = TIGHT ? 1 : 2;
    u32x4 G[PG][GP], S[NSQ][GP][NG];
    f4 nacc[MT][NG];
    auto readG = [&](int q) __attribute__((always_inline)) {
        const uint32_t* gs = smem + (q / MT % GSL) * GSW + lane * 4;
#pragma unroll
        for (int g = 0; g < GP; ++g) G[q % PG][g] = *reinterpret_cast<const u32x4*>(gs + (q % MT * GP + g) * 256);
    };
    // values 2j, 2j + 1 of x*x (1DN: |x|) of pixel tile n0 + nt, pair p, in parts
    auto square = [&](int n0, int p, int nt, int j) __attribute__((always_inline)) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        f2 r;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float x = acc[2 * p + j / 2][n0 + nt][2 * (j % 2) + e];
            r[e] = a.norm1 ? fabsf(x) : x * x;
        }
#pragma unroll
        for (int g = 0; g < GP; ++g) {
            const b2 h = __builtin_convertvector(r, b2);
            S[p % NSQ][g][nt][j] = __builtin_bit_cast(uint32_t, h);
            if (g + 1 < GP) r -= __builtin_convertvector(h, f2);
        }
    };
    // One pair of 16-channel rows of x*x against all of gamma's rows: the
    // products of one row of fragments, the reads of a later one, and a part of
    // the next pair's squares (vector work in the shadow of the products).
    auto pair = [&](auto nc, auto pc_) __attribute__((always_inline)) {
        constexpr int n0 = decltype(nc)::value, p = decltype(pc_)::value;
        constexpr bool landing = n0 == 0 && (RES ? p == 0 || p == HALF : true);              // wait for slices here
        constexpr bool landing_next = p + 1 < NPAIR ? n0 == 0 && (RES ? p + 1 == HALF : true) : true;
        if constexpr (p == 0 || TIGHT) {
#pragma unroll
            for (int nt = 0; nt < NG; ++nt)
#pragma unroll
                for (int j = 0; j < 4; ++j) square(n0, p, nt, j);
        }
        if constexpr (p == 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const f4 b = *reinterpret_cast<const f4*>((CST ? cst + CO : a.beta) + mt * 16 + kg * 4);
#pragma unroll
                for (int nt = 0; nt < NG; ++nt) nacc[mt][nt] = b;
            }
        }
        if constexpr (landing) {
            constexpr int issued = RES ? NPAIR : p == 0 ? GSL : (GSL + p - 1 < NPAIR ? GSL + p - 1 : NPAIR);
            constexpr int needed = RES ? (p == 0 ? HALF : NPAIR) : p + 1;
            wait_vm<(issued - needed) * GW>();
            lds_barrier();
            if constexpr (!RES && p >= 1 && p - 1 + GSL < NPAIR) g_issue(p - 1 + GSL);
        }
        if constexpr (landing || p == 0) {
#pragma unroll
            for (int q = 0; q < PG; ++q) readG(p * MT + q);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const u32x4(&W)[GP] = G[(p * MT + mt) % PG];
            auto mul = [&](int g, int s) __attribute__((always_inline)) {
#pragma unroll
                for (int nt = 0; nt < NG; ++nt)
                    nacc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[g]),
                                                                           __builtin_bit_cast(bf16x8, S[p % NSQ][s][nt]),
                                                                           nacc[mt][nt], 0, 0, 0);
            };
            if constexpr (GP == 3) {
                mul(0, 2);
                mul(1, 1);
                mul(2, 0);
            }
            mul(0, 1);
            mul(1, 0);
            mul(0, 0);
            if (mt + PG < MT || !landing_next) readG(p * MT + mt + PG);
            if (!TIGHT && p + 1 < NPAIR && mt < 4 * NG) square(n0, p + 1, mt / 4, mt % 4);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto group = [&](auto nc) __attribute__((always_inline)) {
        constexpr int n0 = decltype(nc)::value;
        pair(nc, std::integral_constant<int, 0>{});
        pair(nc, std::integral_constant<int, 1>{});
        pair(nc, std::integral_constant<int, 2>{});
        pair(nc, std::integral_constant<int, 3>{});
        static_assert(NPAIR == 4 || NPAIR == 6, "128 or 192 channels");
        if constexpr (NPAIR == 6) {
            pair(nc, std::integral_constant<int, 4>{});
            pair(nc, std::integral_constant<int, 5>{});
        }
        // y = x / sqrt(n) (inverse: x sqrt(n)); 1DN: x / n (x n).  (Row by row: the
        // scheduler would keep every root before the first product.)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < NG; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float nv = nacc[mt][nt][i];
                    if (EP == EP_GDN)
                        acc[mt][n0 + nt][i] *= a.norm1 ? __builtin_amdgcn_rcpf(nv) : __builtin_amdgcn_rsqf(nv);
                    else
                        acc[mt][n0 + nt][i] *= a.norm1 ? nv : __builtin_amdgcn_sqrtf(nv);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    static_assert(NT / NG <= 2, "groups of pixel tiles");
    static_assert(4 * NG <= MT, "a part of the next pair's squares per row");
    group(std::integral_constant<int, 0>{});
    if constexpr (NT > NG) group(std::integral_constant<int, NG>{});
    lds_barrier();                                      // the last slice has been read

    // Each wave writes its pixels' channels to LDS rows and then to memory in
    // 16-byte pieces, consecutive lanes on one pixel; the padding of a row
    // holds the pixel's output offset.
    auto emit = [&](auto oec) __attribute__((always_inline)) {
        constexpr int OE = decltype(oec)::value;        // bytes per stored value
        constexpr int OROW = MT * 16 * OE / 4 + 4;      // words per row
        uint32_t* const ob = smem + wave * (16 * OROW);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint32_t* const row = ob + l16 * OROW;
            const long o = dest(nt);
            if (kg == 0) *reinterpret_cast<long*>(row + MT * 16 * OE / 4) = o;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const f4 v = acc[mt][nt];
                if constexpr (OE == 4) {
                    *reinterpret_cast<f4*>(row + mt * 16 + kg * 4) = v;
                } else if constexpr (OE == 2) {
                    bf16x4 h;
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[i] = (__bf16)v[i];
                    *reinterpret_cast<bf16x4*>(row + mt * 8 + kg * 2) = h;
                } else {
                    const f4 w = a.out_q * v;
                    if (a.sat) {
                        const bool s = o >= 0 && (fabsf(w[0]) > 448.0f || fabsf(w[1]) > 448.0f || fabsf(w[2]) > 448.0f ||
                                                  fabsf(w[3]) > 448.0f);
                        const unsigned long long m = __ballot(s);
                        if (m && lane == __ffsll((long long)m) - 1) atomicAdd(a.sat, (unsigned long long)__popcll(m));
                    }
                    row[mt * 4 + kg] = e4m3x2(w[0], w[1]) | (e4m3x2(w[2], w[3]) << 16);
                }
            }
            wave_order();
            constexpr int PPR = MT * OE;                // 16-byte pieces per pixel
            static_assert(16 * PPR % 64 == 0, "whole stores");
#pragma unroll
            for (int j = 0; j < 16 * PPR / 64; ++j) {
                const int q2 = j * 64 + lane, p2 = q2 / PPR, c = q2 - (q2 / PPR) * PPR;
                const uint32_t* orow = ob + p2 * OROW;
                const long o2 = *reinterpret_cast<const long*>(orow + MT * 16 * OE / 4);
                const u32x4 v = *reinterpret_cast<const u32x4*>(orow + c * 4);
                if (o2 >= 0) *reinterpret_cast<u32x4*>(static_cast<uint8_t*>(a.out) + o2 * OE + c * 16) = v;
            }
            wave_order();
        }
    };
    if constexpr (DT == DT_F32X) {
        emit(std::integral_constant<int, 4>{});
    } else if constexpr (DT == DT_BF16) {
        if (a.out_e4m3) emit(std::integral_constant<int, 1>{});
        else emit(std::integral_constant<int, 2>{});
    } else {
        if (a.out_bf16) emit(std::integral_constant<int, 2>{});
        else emit(std::integral_constant<int, 1>{});
    }
}

}  // namespace lic
