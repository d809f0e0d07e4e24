// Staging in LDS: direct loads from memory, the waits for them, barriers that
// order LDS accesses only, and the scale-table search.
#pragma once
#include <hip/hip_runtime.h>

#include "mfma_common.h"

namespace lic {

// s_waitcnt vmcnt(N) alone (expcnt and lgkmcnt at their maxima)
template <int N> __device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// the same together with lgkmcnt(0): this wave's LDS reads have returned
template <int N> __device__ __forceinline__ void wait_vm_lds()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// workgroup barrier that orders LDS accesses only: loads into LDS that are
// still in flight are waited for by wait_vm where their stage is used (a
// workgroup fence makes the compiler wait for all of them)
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// orders one wave's LDS accesses before and after (lanes read each other's)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A buffer over 2 GiB from a wave-uniform base: loads take a 32-bit lane
// offset (0xffffffff: out of range, reads zero, also into LDS) and a 32-bit
// wave-uniform one, so a moving window costs no vector arithmetic.
#if defined(__HIP_DEVICE_COMPILE__)
using Buf = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Buf make_buf(const void* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00027000);
}
#else                                 // host pass: device types and builtins only
struct Buf {};
__device__ __forceinline__ Buf make_buf(const void*) { return {}; }
#endif
// 16 bytes per lane straight to the 1 KB of LDS at dst (lane l to dst + 16 l; dst
// is the same for every lane)
__device__ __forceinline__ void buf_load_lds(Buf b, uint32_t* dst, uint32_t lane_off, int off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)dst, 16, lane_off, off, 0, 0);
#endif
}
// the same with 4 bytes per lane (lane l to dst + 4 l)
__device__ __forceinline__ void buf_load_lds4(Buf b, uint32_t* dst, uint32_t lane_off, int off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)dst, 4, lane_off, off, 0, 0);
#endif
}
__device__ __forceinline__ u32x4 buf_load(Buf b, uint32_t lane_off, int off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b, lane_off, off, 0));
#else
    return u32x4{0, 0, 0, 0};
#endif
}
// all ones in lane l if bit t of its mask is set, else zero
__device__ __forceinline__ uint32_t bit_mask(uint32_t mask, int t)
{
    return (uint32_t)((int)(mask << (31 - t)) >> 31);
}

// Bit t set: tap t of the window at (oy, ox) falls outside the H x W image, or t
// is past the last tap.  Lane t of tapv holds tap t's offsets (dy low, dx high
// 16 bits).  nx > 0: the taps are rows of nx with one dy each and the same
// dx in every row, so a row and a column test per index decide all of them.
__device__ __forceinline__ uint32_t bad_taps(int oy, int ox, int tapv, int ntaps, int nx, int H, int W)
{
    uint32_t bad = 0xffffffffu << ntaps;
    if (nx > 0) {
        uint32_t col = 0;
        for (int v = 0; v < nx; ++v)
            col |= (unsigned)(ox + (__builtin_amdgcn_readlane(tapv, v) >> 16)) < (unsigned)W ? 0u : 1u << v;
        for (int t = 0; t < ntaps; t += nx) {
            const bool in = (unsigned)(oy + (int)(short)(__builtin_amdgcn_readlane(tapv, t) & 0xffff)) < (unsigned)H;
            bad |= (in ? col : (1u << nx) - 1) << t;
        }
    } else {
        for (int t = 0; t < ntaps; ++t) {
            const int tv = __builtin_amdgcn_readlane(tapv, t);
            const bool in = ((unsigned)(oy + (int)(short)(tv & 0xffff)) < (unsigned)H) & ((unsigned)(ox + (tv >> 16)) < (unsigned)W);
            bad |= in ? 0u : 1u << t;
        }
    }
    return bad;
}

// scale-table index of a pre-activation scale y: #{k < 63 : ts[k] < s} with s
// = y (exp: ts holds ln t_k, exp(y) > t_k <=> y > ln t_k) or s = max(y, 0, t_0)
// (ts holds t_k).  The table is log-spaced, so (s - ts[0]) / step (ReLU:
// log2(s / ts[0]) / step) is within a step or two of the count; from there
// it is settled by comparisons with the table itself, so the result is
// exactly the count whatever the first guess.
__device__ __forceinline__ int scale_count(float y, const float* ts, float t0, float inv, int hs_exp)
{
    const float s = hs_exp ? y : fmaxf(fmaxf(y, 0.0f), t0);
    const float u = hs_exp ? (s - t0) * inv : (__log2f(s) - __log2f(t0)) * inv;
    int e = (int)ceilf(fminf(fmaxf(u, 0.0f), 63.0f));     // NaN: 0
    while (e < 63 && ts[e] < s) ++e;
    while (e > 0 && !(ts[e - 1] < s)) --e;
    return e;
}

}  // namespace lic
