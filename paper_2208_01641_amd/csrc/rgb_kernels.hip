// g_s's output layer on MFMA (gfx950): a stride-2 transposed convolution to 3
// channels as 12 GEMM rows (4 sub-pixel phases x 3 channels) over the 3 x 3
// neighbourhood of each grid position, then the clamp and the crop.
//
// A block covers 8 x 32 grid positions (every grid is a multiple of that), a
// wave 2 rows of 32.  Per channel slice (64 bytes a position) the 10 x 34 halo
// tile and the slice's nine weight fragments go straight from memory to LDS,
// one slice ahead; positions outside the image read zero from beyond the
// buffer's range.  FP32 products share the vector pipe with every other vector
// instruction, so the loop has none: a tap is a constant offset from one of
// three lane addresses (the rows' pitch is a multiple of 8 positions, so the
// rotation that spreads a position's four pieces over the banks depends on the
// column alone).  Outputs are transposed in LDS and leave as whole rows.
// The products and their order are those of conv_igemm's halo tiles.
//
// 720p, kernel time (us), before -> now: FP32 109 -> 87 (2.4 GHz of products alone:
// 61, at the clock the chip holds under them about 69; reading a tap's fragments
// one tap ahead by hand changed nothing), bf16 34 -> 24.  FP32 operands split into
// three bf16 parts took 59 us and are not used: one product by itself was then up
// to 2.9 x 2^-24 off (here 1.0), and a finite activation that bf16 rounds to
// infinity gave NaN.
#include <hip/hip_runtime.h>

#include "../../include/lic.h"
#include "conv_args.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

template <int CIN, int DT>
__global__ void __launch_bounds__(256, 2) rgb_tile(ConvArgs a)
{
    static_assert(DT == DT_F32 || DT == DT_BF16, "FP32 or bf16 operands");
    constexpr int KCH = Prec<DT>::KCH;                  // 64 bytes of a position
    constexpr int ESZ = (int)sizeof(typename Prec<DT>::Elem);
    constexpr int NS = CIN / KCH;                       // channel slices
    constexpr int TH = 8, TW = 32, PITCH = 40, HR = TH + 2;
    constexpr int PI = HR * PITCH / 16, NI = PI + 9;    // 1 KB loads per slice: positions, weights
    constexpr int IW = (NI + 3) / 4;                    // loads per wave (past the end: the last again)
    constexpr int STW = NI * 256;                       // words per stage
    static_assert(HR * PITCH % 16 == 0 && PITCH % 8 == 0 && PITCH >= TW + 2, "tile layout");
    constexpr int OW = 2 * TW + 1;                      // words per staged output row
    static_assert(3 * 2 * TH * OW <= 2 * STW, "output rows fit the stages");
    __shared__ __attribute__((aligned(16))) uint32_t smem[2 * STW];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int logical = xcd_logical_tile(blockIdx.x, gridDim.x);
    const int bx = a.Wg / TW, by = a.Hg / TH;
    const int img = logical / (bx * by), rem = logical - img * (bx * by);
    const int ty = (rem / bx) * TH, tx = (rem - (rem / bx) * bx) * TW;

    // this lane's piece in each of the wave's loads, from the tile's first row
    // (0xffffffff: outside the image, or padding of the pitch)
    const uint8_t* const in0 = static_cast<const uint8_t*>(a.in) + ((long)img * a.Hin + ty) * a.Win * (long)(CIN * ESZ);
    const Buf ibuf = make_buf(in0 - (long)a.Win * (CIN * ESZ));        // one row up
    const Buf wbuf = make_buf(static_cast<const uint8_t*>(a.ws) + a.ph->wtoff * ESZ);
    uint32_t off[IW];
#pragma unroll
    for (int u = 0; u < IW; ++u) {
        const int f = min(wave * IW + u, NI - 1);
        const int pos = f * 16 + lane / 4, hr = pos / PITCH, hc = pos - hr * PITCH;
        const int y = ty + hr - 1, x = tx + hc - 1;
        const bool in = hc < TW + 2 && (unsigned)y < (unsigned)a.Hin && (unsigned)x < (unsigned)a.Win;
        const int piece = (lane & 3) ^ ((hc >> 1) & 3);
        off[u] = f >= PI ? (uint32_t)(lane * 16) : in ? (uint32_t)((hr * a.Win + x) * (CIN * ESZ) + piece * 16) : 0xffffffffu;
    }
    auto issue = [&](int s, uint32_t* st) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < IW; ++u) {
            const int f = min(wave * IW + u, NI - 1);
            if (f >= PI) buf_load_lds(wbuf, st + f * 256, off[u], (s * 9 + f - PI) * 1024);
            else buf_load_lds(ibuf, st + f * 256, off[u], s * 64);
        }
    };

    f4 acc[4];
    {
        const f4 b = *reinterpret_cast<const f4*>(a.bias + kg * 4);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[nt] = b;
    }
    // lane addresses (words) of the columns dx = -1, 0, 1 of this wave's first row
    int col[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int hc = l16 + d;
        col[d] = (wave * 2 * PITCH + hc) * 16 + ((kg ^ ((hc >> 1) & 3)) * 4);
    }
    issue(0, smem);
#pragma unroll 1
    for (int s = 0; s < NS; ++s) {
        const uint32_t* const st = smem + (s & 1) * STW;
        wait_vm<0>();
        lds_barrier();                                  // slice s is here, slice s - 1 has been read
        if (s + 1 < NS) issue(s + 1, smem + ((s + 1) & 1) * STW);
        const uint32_t* const c[3] = {st + col[0], st + col[1], st + col[2]};
        const uint32_t* const w = st + PI * 256 + lane * 4;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const u32x4 A = *reinterpret_cast<const u32x4*>(w + t * 256);
            u32x4 B[4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)              // row nt / 2, columns 16 (nt % 2) ..
                B[nt] = *reinterpret_cast<const u32x4*>(c[t % 3] + ((t / 3 + nt / 2) * PITCH + (nt % 2) * 16) * 16);
            if constexpr (DT == DT_F32) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
                        acc[nt] = mfma16x16x4(__builtin_bit_cast(f4, A)[e], __builtin_bit_cast(f4, B[nt])[e], acc[nt]);
            } else {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A),
                                                                      __builtin_bit_cast(bf16x8, B[nt]), acc[nt], 0, 0, 0);
            }
        }
    }

    // rows r = 3 (2 py + px) + c of position (y, x): channel c of pixel (2y + py, 2x + px)
    lds_barrier();
    float* const o = reinterpret_cast<float*>(smem);    // [3][2 TH][OW]
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = kg * 4 + i, q = r / 3, c = r - 3 * q;
            const int row = 2 * (wave * 2 + nt / 2) + (q >> 1), x = 2 * ((nt % 2) * 16 + l16) + (q & 1);
            if (r < 12) o[(c * 2 * TH + row) * OW + x] = acc[nt][i];
        }
    lds_barrier();
    float* const out = static_cast<float*>(a.out);
    float* const pre = static_cast<float*>(a.aux);
    const int x = 2 * tx + lane;
    for (int j = wave; j < 3 * 2 * TH; j += 4) {
        const int c = j / (2 * TH), y = 2 * ty + j - c * 2 * TH;
        const float v = o[j * OW + lane];
        if (pre) pre[(((long)img * 3 + c) * a.Hout + y) * a.Wout + x] = v;
        if (out && y < a.Hc && x < a.Wc) out[(((long)img * 3 + c) * a.Hc + y) * a.Wc + x] = fminf(fmaxf(v, 0.0f), 1.0f);
    }
}

bool rgb_available(int cin, int dt) { return (cin == 128 || cin == 192) && (dt == DT_F32 || dt == DT_BF16); }

hipError_t launch_rgb(int cin, int dt, const ConvArgs& a, hipStream_t stream)
{
    const dim3 grid(a.n * (a.Hg / 8) * (a.Wg / 32));
    if (dt == DT_F32)
        hipLaunchKernelGGL(cin == 128 ? (rgb_tile<128, DT_F32>) : (rgb_tile<192, DT_F32>), grid, dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(cin == 128 ? (rgb_tile<128, DT_BF16>) : (rgb_tile<192, DT_BF16>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace lic
