// Device helpers shared by the convolution kernels: operand types of the
// four GEMM forms, the bf16 splitting of FP32 values, e4m3 conversion and the
// XCD-aware block order.
#pragma once
#include <hip/hip_runtime.h>

#include "conv_args.h"

namespace lic {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma16x16x4(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Operand precision of the convolution GEMM (accumulation is always FP32).
//   DT_F32 : v_mfma_f32_16x16x4_f32, 16-channel K chunks, 4 channels per lane
//   DT_BF16: v_mfma_f32_16x16x32_bf16, 32-channel K chunks, 8 channels per
//            lane (one 16-byte load); activations between layers are stored
//            as bf16, GDN / IGDN and all epilogue arithmetic stay FP32.
template <int DT> struct Prec;
// Frag: weight (A) fragment of one lane and K chunk; BIn: pixel (B) values
// as loaded from NHWC activations; BFrag: B as fed to the matrix cores;
// Elem / WElem: activation / weight element; WMUL: weight elements per
// weight value.
template <> struct Prec<DT_F32> {
    using Frag = f4;
    using Elem = float;
    using WElem = float;
    using BIn = f4;
    using BFrag = f4;
    static constexpr int KCH = 16, KE = 4, WMUL = 1;
};
template <> struct Prec<DT_BF16> {
    using Frag = bf16x8;
    using Elem = __bf16;
    using WElem = __bf16;
    using BIn = bf16x8;
    using BFrag = bf16x8;
    static constexpr int KCH = 32, KE = 8, WMUL = 1;
};
//   DT_F32X: FP32 operands split exactly into three bf16 parts (each rounded
//            to nearest from what the previous parts leave: v = v0 + v1 + v2
//            up to 2^-27 |v|); the products of parts i + j <= 2 run on
//            v_mfma_f32_16x16x32_bf16 (each exact in FP32) with FP32
//            accumulation, so a product is at most 3 x 2^-24 off (2 of it what
//            the products left out can hold), most near 2^-25.  Weights are split on the host
//            ([part][8] per 8 channels), activations stay FP32 and are split
//            when a chunk is used.
struct Split3 {
    bf16x8 p[3];
};
struct F32x8 {
    f4 lo, hi;
};
template <> struct Prec<DT_F32X> {
    using Frag = Split3;
    using Elem = float;
    using WElem = __bf16;
    using BIn = F32x8;
    using BFrag = Split3;
    static constexpr int KCH = 32, KE = 8, WMUL = 3;
};
//   DT_FP8 : v_mfma_scale_f32_16x16x128_f8f6f4 on OCP e4m3 operands (unit
//            block scales), K walked over the flattened (tap, channel) axis in
//            chunks of 128: lane group g takes 32 consecutive channels of one
//            tap (channels per tap are a multiple of 32).  Weights carry a
//            per-row FP32 scale and activations are stored as e4m3(q x) with
//            a per-layer q, both undone in the epilogue; the operands come
//            from e4m3 activations only (the image layer and g_s's first and
//            last layers of that form run on bf16 operands).
template <> struct Prec<DT_FP8> {
    using Frag = i32x8;
    using Elem = uint8_t;
    using WElem = uint8_t;
    using BIn = i32x8;
    using BFrag = i32x8;
    static constexpr int KCH = 128, KE = 32, WMUL = 1;
};

// eight FP32 values as G bf16 parts, each rounded to nearest (v_cvt_pk_bf16_f32,
// two values per instruction) from what the previous parts leave, which is
// exact in FP32: v = v0 + ... + v_{G-1} up to the rounding of the last part
template <int G>
__device__ __forceinline__ void split_parts(const float (&v)[8], bf16x8 (&out)[G])
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    u32x4 w[G];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f2 r = {v[2 * j], v[2 * j + 1]};
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const b2 h = __builtin_convertvector(r, b2);
            w[g][j] = __builtin_bit_cast(uint32_t, h);
            if (g + 1 < G) r -= __builtin_convertvector(h, f2);
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) out[g] = __builtin_bit_cast(bf16x8, w[g]);
}

// eight FP32 values as three bf16 parts (v = v0 + v1 + v2 up to 2^-27 |v|)
__device__ __forceinline__ Split3 split3(const float (&v)[8])
{
    Split3 s;
    split_parts<3>(v, s.p);
    return s;
}

// e4m3 code of two floats in the low 16 bits, saturated to +-448 first
__device__ __forceinline__ uint32_t e4m3x2(float lo, float hi)
{
    lo = fminf(fmaxf(lo, -448.0f), 448.0f);
    hi = fminf(fmaxf(hi, -448.0f), 448.0f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(lo, hi, 0, false) & 0xffffu;
}

// unit E8M0 block scale (2^0) of the scaled MFMA
constexpr int kE8M0One = 127;

// Blocks are dispatched round-robin over the 8 XCDs (block L goes to XCD
// L % 8).  Give each XCD a contiguous range of logical tiles so that tiles
// sharing input halos and weights share one L2.
__device__ __forceinline__ int xcd_logical_tile(int L, int T)
{
    const int xcd = L & 7, slot = L >> 3;
    int prefix = 0;
    for (int q = 0; q < xcd; ++q) prefix += (T + 7 - q) >> 3;
    return prefix + slot;
}

}  // namespace lic
