// g_s's output layer on MFMA (gfx950): a stride-2 transposed convolution to 3
// channels as 12 GEMM rows (4 sub-pixel phases x 3 channels) over the 3 x 3
// neighbourhood of each grid position, then the clamp and the crop.
//
// bf16 form (rgb_tile): a block covers 8 x 32 grid positions (every grid is a
// multiple of that), a wave 2 rows of 32.  Per channel slice (64 bytes a
// position) the 10 x 34 halo tile and the slice's nine weight fragments go
// straight from memory to LDS, one slice ahead; positions outside the image
// read zero from beyond the buffer's range.  A tap is a constant offset from one
// of three lane addresses (the rows' pitch is a multiple of 8 positions, so the
// rotation that spreads a position's four pieces over the banks depends on the
// column alone).  Outputs are transposed in LDS and leave as whole rows.  The
// products and their order are those of conv_igemm's halo tiles.  720p: 34 -> 24 us
// of kernel time.
//
// FP32 form (rgb_split): operands split in three bf16 parts.  FP32 products
// hold this layer at 87 us (720p; 61 of products alone at 2.4 GHz): 16 positions
// take 288 of them, 32 clocks each, against 216 bf16 products of 16 clocks.
// Kernel time 87 -> 59 us, 128 x 128 24 -> 11; what bounds it is LDS (a wave's 27
// weight fragments and 36 of positions per slice serve 108 products) with the
// products close behind; reading the input takes 26 us at the rate of a copy.  Error
// against 64 bits (2-norm) at 720p: FP32 products 6.3e-7, here 2.0e-7.
#include <hip/hip_runtime.h>

#include "../../include/lic.h"
#include "conv_args.h"
#include "kernels.h"
#include "lds_stage.h"
#include "mfma_common.h"

namespace lic {

template <int CIN>
__global__ void __launch_bounds__(256, 2) rgb_tile(ConvArgs a)
{
    constexpr int DT = DT_BF16;
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
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A),
                                                                  __builtin_bit_cast(bf16x8, B[nt]), acc[nt], 0, 0, 0);
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

// A position is split once, when its slice is staged (splitting fragments per
// tap would cost more than the products): loads go to registers during the
// previous slice's products, four lanes to a 64-byte run (so a lane group has
// four channels of either half of the slice), and the parts to three planes in LDS,
// 64 bytes a position and rotated by column as above.  A block covers 8 x 16
// positions, a wave RW rows of them; a window row's fragments serve the three taps
// of a column that meet it.  (16 x 32 positions and 8 waves, one block per CU: 60 us
// at 720p, 26 against 18 at 360p, 23 against 11 at 128 x 128.)  The products of the
// first parts have sums of their own, the small products others, added at the end:
// fewer roundings in the large sum.  An infinite activation, or one that bf16
// rounds to infinity, gives NaN, as in the other split layers.
template <int CIN>
__global__ void __launch_bounds__(256, 2) rgb_split(ConvArgs a)
{
    constexpr int NS = CIN / 32, WAVES = 4, THREADS = 64 * WAVES, RW = 2;
    constexpr int TH = WAVES * RW, TW = 16, WP = TW + 2, WPX = (TH + 2) * WP;
    constexpr int PL = WPX * 16;                        // words per plane (one part)
    constexpr int AF = 27, AW = (AF + WAVES - 1) / WAVES;   // weight fragments per slice, of a wave
    constexpr int UN = (WPX * 4 + THREADS - 1) / THREADS;   // 8-channel pieces per thread and slice
    constexpr int OW = 2 * TW + 1;
    constexpr int SMW = 3 * PL + AF * 256;
    static_assert(SMW * 4 <= 81920, "two blocks per CU");
    static_assert(3 * 2 * TH * OW <= SMW, "output rows fit");
    __shared__ __attribute__((aligned(16))) uint32_t smem[SMW];
    uint32_t* const sw = smem + 3 * PL;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int logical = xcd_logical_tile(blockIdx.x, gridDim.x);
    const int bx = a.Wg / TW, by = a.Hg / TH;
    const int img = logical / (bx * by), rem = logical - img * (bx * by);
    const int ty = (rem / bx) * TH, tx = (rem - (rem / bx) * bx) * TW;
    const Buf ibuf = make_buf(static_cast<const float*>(a.in) + ((long)img * a.Hin + ty - 1) * a.Win * (long)CIN);
    const Buf wbuf = make_buf(static_cast<const uint8_t*>(a.ws) + a.ph->wtoff * 6);

    uint32_t off[UN];
    int dst[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        const int q = min(u * THREADS + (int)threadIdx.x, WPX * 4 - 1);      // (past the end: the last again)
        const int px = q >> 2, c = q & 3, r = px / WP, col = px - r * WP;
        const bool in = (unsigned)(ty + r - 1) < (unsigned)a.Hin && (unsigned)(tx + col - 1) < (unsigned)a.Win;
        off[u] = in ? (uint32_t)((r * a.Win + tx + col - 1) * (CIN * 4) + c * 16) : 0xffffffffu;
        dst[u] = px * 16 + ((c ^ ((col >> 1) & 3)) * 4);
    }
    u32x4 X[UN][2];
    auto load = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) X[u][h] = buf_load(ibuf, off[u], s * 128 + h * 64);
    };
    int col[3];                                         // words to columns dx = -1, 0, 1 of the wave's first window row
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int cc = l16 + d;
        col[d] = (wave * RW * WP + cc) * 16 + ((kg ^ ((cc >> 1) & 3)) * 4);
    }
    f4 hi[RW], lo[RW];
#pragma unroll
    for (int y = 0; y < RW; ++y) {
        hi[y] = *reinterpret_cast<const f4*>(a.bias + kg * 4);
        lo[y] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    load(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s > 0) lds_barrier();                       // slice s - 1 has been read
#pragma unroll
        for (int u = 0; u < AW; ++u) {
            const int f = min(wave * AW + u, AF - 1);
            buf_load_lds(wbuf, sw + f * 256, lane * 16, (s * AF + f) * 1024);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const f4 x0 = __builtin_bit_cast(f4, X[u][0]), x1 = __builtin_bit_cast(f4, X[u][1]);
            const float v[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
            const Split3 p = split3(v);
#pragma unroll
            for (int g = 0; g < 3; ++g) *reinterpret_cast<u32x4*>(smem + dst[u] + g * PL) = __builtin_bit_cast(u32x4, p.p[g]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < NS) load(s + 1);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < NS) wait_vm<2 * UN>();
        else wait_vm<0>();
        lds_barrier();                                  // positions and weights of the slice are here
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            bf16x8 A[3][3];
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int g = 0; g < 3; ++g)
                    A[t][g] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sw + ((t * 3 + d) * 3 + g) * 256 + lane * 4));
#pragma unroll
            for (int r = 0; r < RW + 2; ++r) {
                bf16x8 B[3];
#pragma unroll
                for (int g = 0; g < 3; ++g)
                    B[g] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(smem + col[d] + r * (WP * 16) + g * PL));
                constexpr int pa[6] = {0, 1, 2, 0, 1, 0}, pb[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
                for (int m = 0; m < 6; ++m)
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const int y = r - t;
                        if (y < 0 || y >= RW) continue;
                        f4& c = m == 5 ? hi[y] : lo[y];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t][pa[m]], B[pb[m]], c, 0, 0, 0);
                    }
            }
        }
    }

    // rows r = 3 (2 py + px) + c of position (y, x): channel c of pixel (2y + py, 2x + px)
    lds_barrier();
    float* const o = reinterpret_cast<float*>(smem);    // [3][2 TH][OW]
#pragma unroll
    for (int y = 0; y < RW; ++y)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = kg * 4 + i, q = r / 3, c = r - 3 * q;
            const int row = 2 * (wave * RW + y) + (q >> 1), x = 2 * l16 + (q & 1);
            if (r < 12) o[(c * 2 * TH + row) * OW + x] = hi[y][i] + lo[y][i];
        }
    lds_barrier();
    float* const out = static_cast<float*>(a.out);
    float* const pre = static_cast<float*>(a.aux);
    for (int j = threadIdx.x; j < 3 * 2 * TH * 2 * TW; j += THREADS) {
        const int row = j / (2 * TW), x = 2 * tx + j - row * (2 * TW);
        const int c = row / (2 * TH), y = 2 * ty + row - c * 2 * TH;
        const float v = o[row * OW + x - 2 * tx];
        if (pre) pre[(((long)img * 3 + c) * a.Hout + y) * a.Wout + x] = v;
        if (out && y < a.Hc && x < a.Wc) out[(((long)img * 3 + c) * a.Hc + y) * a.Wc + x] = fminf(fmaxf(v, 0.0f), 1.0f);
    }
}

bool rgb_available(int cin, int dt) { return (cin == 128 || cin == 192) && (dt == DT_F32 || dt == DT_BF16); }

hipError_t launch_rgb(int cin, int dt, const ConvArgs& a, hipStream_t stream)
{
    const long positions = (long)a.n * a.Hg * a.Wg;
    if (dt == DT_F32)
        hipLaunchKernelGGL(cin == 128 ? rgb_split<128> : rgb_split<192>, dim3((unsigned)(positions / 128)), dim3(256), 0,
                           stream, a);
    else
        hipLaunchKernelGGL(cin == 128 ? rgb_tile<128> : rgb_tile<192>, dim3((unsigned)(positions / 256)), dim3(256), 0,
                           stream, a);
    return hipGetLastError();
}

}  // namespace lic
