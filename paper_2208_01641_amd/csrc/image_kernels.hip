// g_a's first layer on MFMA (gfx950): image ingest (NCHW float, zero padding),
// 5 x 5 stride-2 convolution to 128 channels and GDN.
//
// Its convolution is short (75 products a channel), so what bounds it is
// everything else: gathering pixels one float at a time, the contraction over
// channels (four fifths of the products), and getting 128 channels a pixel out.
// One block of 8 waves per CU stays for its whole share of the grid:
//   * gamma (bf16 form: and the weights) sits in LDS for good, so the loop has no
//     barrier and the waves drift apart, one's loads under another's products;
//   * a wave takes 32 pixels of one row: the window (3 x 5 x 67 floats) goes
//     straight from memory to LDS in whole rows, the next one as soon as the
//     operands of this one are in registers; outside the image the loads are
//     out of the buffer's range and read zero;
//   * outputs are transposed in LDS and leave in 16-byte pieces.
// (streaming stores: no change, neither here nor in the whole codec)
// Products and sums are those of conv_igemm: k = (5 u + v) 3 + c in three
// chunks of 32, then n = beta + gamma (x*x).
//
// 720p, kernel time (us), before -> now: split-FP32 107 -> 77 (matrix cores busy
// 43% of it; 127 MB of output), bf16 74 -> 42, e4m3 76 -> 48.
#include <hip/hip_runtime.h>

#include "../../include/lic.h"
#include "conv_args.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

template <int DT>
__global__ void __launch_bounds__(512, 1) image_gdn(ConvArgs a)
{
    static_assert(DT == DT_F32X || DT == DT_BF16, "split-FP32 or bf16 operands");
    constexpr int MT = 8, NT = 2, WAVES = 8, NPAIR = MT / 2;
    constexpr int GP = DT == DT_F32X ? 3 : 2;           // bf16 parts of gamma and x*x
    constexpr int CROW = 68, CW = 384;                  // window: floats per row, per channel (5 rows, then zeros)
    constexpr int CI = CW / 64;                         // loads per channel
    constexpr int WW = 3 * CW;                          // words per wave's window
    constexpr int AWORDS = DT == DT_BF16 ? 3 * MT * 256 : 0;
    constexpr int GWORDS = NPAIR * MT * GP * 256;
    // staged output: 16 pixels x SC channels (plus 16 bytes a row)
    constexpr int SC = DT == DT_F32X ? 32 : 128;
    constexpr int ORMAX = (DT == DT_F32X ? SC : SC / 2) + 4;
    constexpr int OWORDS = 16 * ORMAX;
    constexpr int BW = 2 * MT * 16;                     // bias, beta
    constexpr int SMW = AWORDS + GWORDS + WAVES * (WW + OWORDS) + BW;
    static_assert(SMW * 4 <= 163840, "one block per CU");
    __shared__ __attribute__((aligned(16))) uint32_t smem[SMW];
    uint32_t* const sA = smem;
    uint32_t* const sG = smem + AWORDS;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    uint32_t* const win = smem + AWORDS + GWORDS + wave * WW;
    uint32_t* const ob = smem + AWORDS + GWORDS + WAVES * WW + wave * OWORDS;

    // (bias and beta in LDS too: a load from memory in the loop would wait for the
    // next window, which is on its way before it)
    float* const sB = reinterpret_cast<float*>(smem + AWORDS + GWORDS + WAVES * (WW + OWORDS));
    if (threadIdx.x < BW) sB[threadIdx.x] = threadIdx.x < MT * 16 ? a.bias[threadIdx.x] : a.beta[threadIdx.x - MT * 16];
    const Buf wbuf = make_buf(a.ws), gbuf = make_buf(a.gt);
    for (int f = wave; f < AWORDS / 256; f += WAVES) buf_load_lds(wbuf, sA + f * 256, lane * 16, f * 1024);

    // tiles of 32 pixels (a row holds whole ones): this block's share, one in
    // 8 of it per wave
    const int tw = a.Wg / 32, HWt = a.Hg * tw, ntile = a.n * HWt;
    const int lb = xcd_logical_tile(blockIdx.x, gridDim.x);
    const int t_end = (int)((long)(lb + 1) * ntile / gridDim.x);
    int t = (int)((long)lb * ntile / gridDim.x) + wave;

    // window load i of a channel: this lane's float (row u, column j)
    int wu[CI], wj[CI];
#pragma unroll
    for (int i = 0; i < CI; ++i) {
        const int f = i * 64 + lane;
        wu[i] = f / CROW;
        wj[i] = f - wu[i] * CROW;
    }
    auto window = [&](int tile) __attribute__((always_inline)) {
        const int im = tile / HWt, r = tile - im * HWt, gy = r / tw, gx = (r - gy * tw) * 32;
        const int iy = 2 * gy - 2, ix = 2 * gx - 2;
        uint32_t off[CI];
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            const bool in = wu[i] < 5 && wj[i] < CROW - 1 && (unsigned)(iy + wu[i]) < (unsigned)a.Hin &&
                            (unsigned)(ix + wj[i]) < (unsigned)a.Win;
            // (from the image's start of row iy: never below the buffer's base where it is read)
            off[i] = in ? (uint32_t)((wu[i] * a.Win + wj[i]) * 4) : 0xffffffffu;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Buf b = make_buf(static_cast<const float*>(a.in) + (((long)im * 3 + c) * a.Hin + iy) * a.Win + ix);
#pragma unroll
            for (int i = 0; i < CI; ++i) buf_load_lds4(b, win + c * CW + i * 64, off[i], 0);
        }
    };
    // operand k of this lane group: its float in the window (past 3 x 25: a zero)
    int ko[3][8];
#pragma unroll
    for (int kc = 0; kc < 3; ++kc)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = kc * 32 + kg * 8 + e, tap = k / 3, c = k - 3 * tap, u = tap / 5;
            ko[kc][e] = k < 75 ? c * CW + u * CROW + (tap - 5 * u) + 2 * l16 : 2 * CW + 5 * CROW;
        }
    if (t < t_end) window(t);
    // gamma comes last: the first tile is multiplied before it is waited for
    constexpr int GI = GWORDS / 256 / WAVES;
    static_assert(GWORDS / 256 % WAVES == 0, "whole loads per wave");
#pragma unroll
    for (int f = 0; f < GI; ++f) buf_load_lds(gbuf, sG + (f * WAVES + wave) * 256, lane * 16, (f * WAVES + wave) * 1024);
    wait_vm<GI>();
    __syncthreads();                                    // bias, beta and the weights are in LDS
    bool gamma_here = false;                            // (the same for every wave of the block at each barrier)

    for (; t < t_end; t += WAVES) {
        // (the stores of the previous tile, issued after this window, may still be on their way)
        if constexpr (DT == DT_F32X) wait_vm<16>();
        else if (a.out_e4m3) wait_vm<4>();
        else wait_vm<8>();
        wave_order();
        auto operands = [&](int kc, float (&v)[NT][8]) __attribute__((always_inline)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[nt][e] = __builtin_bit_cast(float, win[ko[kc][e] + nt * 32]);
        };
        // the next window, once this one has been read (the weights that the
        // split-FP32 form loads from memory come back in order: before it)
        auto next = [&]() __attribute__((always_inline)) {
            wait_vm_lds<63>();
            __builtin_amdgcn_sched_barrier(0);
            if (t + WAVES < t_end) window(t + WAVES);
        };
        bf16x8 Bh[3][NT];
        if constexpr (DT == DT_BF16) {
#pragma unroll
            for (int kc = 0; kc < 3; ++kc) {
                float v[NT][8];
                operands(kc, v);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 8; ++e) Bh[kc][nt][e] = (__bf16)v[nt][e];
            }
            next();
        }

        f4 acc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f4 b = *reinterpret_cast<const f4*>(sB + mt * 16 + kg * 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = b;
        }
        if constexpr (DT == DT_F32X) {
            constexpr int PF = 4;                       // weight fragments in flight (three parts each)
            u32x4 A[PF][3];
            auto load = [&](int q) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < 3; ++g) A[q % PF][g] = buf_load(wbuf, lane * 16 + g * 1024, q * 3072);
            };
#pragma unroll
            for (int q = 0; q < PF; ++q) load(q);
            float v[NT][8];
            operands(0, v);
#pragma unroll
            for (int kc = 0; kc < 3; ++kc) {
                Split3 Bx[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) Bx[nt] = split3(v[nt]);
                if (kc < 2) operands(kc + 1, v);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int q = kc * MT + mt;
                    constexpr int pa[6] = {0, 1, 2, 0, 1, 0}, pbx[6] = {2, 1, 0, 1, 0, 0};   // smallest first
#pragma unroll
                    for (int s = 0; s < 6; ++s)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[q % PF][pa[s]]),
                                                                                  Bx[nt].p[pbx[s]], acc[mt][nt], 0, 0, 0);
                    if (q + PF < 3 * MT) load(q + PF);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            next();
        } else {
#pragma unroll
            for (int kc = 0; kc < 3; ++kc)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const bf16x8 A = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sA + (kc * MT + mt) * 256 + lane * 4));
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, Bh[kc][nt], acc[mt][nt], 0, 0, 0);
                }
        }

        if (!gamma_here) {
            wait_vm<0>();
            lds_barrier();
            gamma_here = true;
        }
        f4 nacc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f4 b = *reinterpret_cast<const f4*>(sB + MT * 16 + mt * 16 + kg * 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) nacc[mt][nt] = b;
        }
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) {
            bf16x8 S[GP][NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float r[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float x = acc[2 * p + i / 4][nt][i % 4];
                    r[i] = a.norm1 ? fabsf(x) : x * x;
                }
                bf16x8 parts[GP];
                split_parts<GP>(r, parts);
#pragma unroll
                for (int g = 0; g < GP; ++g) S[g][nt] = parts[g];
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                bf16x8 G[GP];
#pragma unroll
                for (int g = 0; g < GP; ++g)
                    G[g] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sG + ((p * MT + mt) * GP + g) * 256 + lane * 4));
                auto mul = [&](int g, int s) __attribute__((always_inline)) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        nacc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G[g], S[s][nt], nacc[mt][nt], 0, 0, 0);
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
        }

        // the tile's pixels follow each other in the output (all of one row)
        const int im = t / HWt, r = t - im * HWt, gy = r / tw, gx = (r - gy * tw) * 32;
        const long opix = ((long)im * a.Hout + gy) * a.Wout + gx;
        auto emit = [&](auto oec) __attribute__((always_inline)) {
            constexpr int OE = decltype(oec)::value;    // bytes per stored value
            constexpr int OROW = SC * OE / 4 + 4;
            constexpr int PPR = SC * OE / 16;           // 16-byte pieces of a staged row
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int m0 = 0; m0 < MT; m0 += SC / 16) {
#pragma unroll
                    for (int m = 0; m < SC / 16; ++m) {
                        const int mt = m0 + m;
                        f4 y;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float nv = nacc[mt][nt][i];
                            y[i] = acc[mt][nt][i] * (a.norm1 ? __builtin_amdgcn_rcpf(nv) : __builtin_amdgcn_rsqf(nv));
                        }
                        uint32_t* const row = ob + l16 * OROW;
                        if constexpr (OE == 4) {
                            *reinterpret_cast<f4*>(row + m * 16 + kg * 4) = y;
                        } else if constexpr (OE == 2) {
                            bf16x4 h;
#pragma unroll
                            for (int i = 0; i < 4; ++i) h[i] = (__bf16)y[i];
                            *reinterpret_cast<bf16x4*>(row + m * 8 + kg * 2) = h;
                        } else {
                            const f4 w = a.out_q * y;
                            if (a.sat) {
                                const bool s = fabsf(w[0]) > 448.0f || fabsf(w[1]) > 448.0f || fabsf(w[2]) > 448.0f ||
                                               fabsf(w[3]) > 448.0f;
                                const unsigned long long mk = __ballot(s);
                                if (mk && lane == __ffsll((long long)mk) - 1) atomicAdd(a.sat, (unsigned long long)__popcll(mk));
                            }
                            row[m * 4 + kg] = e4m3x2(w[0], w[1]) | (e4m3x2(w[2], w[3]) << 16);
                        }
                    }
                    wave_order();
                    uint8_t* const dst = static_cast<uint8_t*>(a.out) + ((opix + nt * 16) * (MT * 16) + m0 * 16) * OE;
#pragma unroll
                    for (int j = 0; j < 16 * PPR / 64; ++j) {
                        const int q = j * 64 + lane, p = q / PPR, c = q - (q / PPR) * PPR;
                        *reinterpret_cast<u32x4*>(dst + p * (MT * 16 * OE) + c * 16) =
                            *reinterpret_cast<const u32x4*>(ob + p * OROW + c * 4);
                    }
                    wave_order();
                }
        };
        if constexpr (DT == DT_F32X) {
            emit(std::integral_constant<int, 4>{});
        } else {
            if (a.out_e4m3) emit(std::integral_constant<int, 1>{});
            else emit(std::integral_constant<int, 2>{});
        }
    }
    if (!gamma_here) {                                  // a wave without a tile brings its part of gamma
        wait_vm<0>();
        lds_barrier();
    }
}

// (192 channels: gamma alone takes 216 KB in three parts, 144 KB in two beside 36 KB
// of weights and the windows; a CU has 160.)
bool image_available(int cop, int dt) { return cop == 128 && (dt == DT_F32X || dt == DT_BF16); }

hipError_t launch_image(int dt, const ConvArgs& a, hipStream_t stream)
{
    const long ntile = (long)a.n * a.Hg * (a.Wg / 32);
    const dim3 grid((unsigned)(ntile < 256 ? ntile : 256));
    if (dt == DT_F32X) hipLaunchKernelGGL(image_gdn<DT_F32X>, grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL(image_gdn<DT_BF16>, grid, dim3(512), 0, stream, a);
    return hipGetLastError();
}

}  // namespace lic
