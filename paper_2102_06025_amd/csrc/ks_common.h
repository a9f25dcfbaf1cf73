// Shared device/host helpers of the KNN-softmax HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/knnsoftmax.h"

#define KS_WAVE 64

// ----- host helpers ---------------------------------------------------------------------------
static inline size_t ks_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int64_t ks_ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// bump allocator over the caller's workspace; every block 256-byte aligned
struct KsArena {
    char *base;
    size_t off;
    explicit KsArena(void *p) : base((char *)p), off(0) {}
    template <typename T> T *take(size_t n) {
        T *r = (T *)(base ? base + off : nullptr);
        off += ks_align_up(n * sizeof(T), 256);
        return r;
    }
};

#define KS_LAUNCH_CHECK()                                  \
    do {                                                   \
        if (hipGetLastError() != hipSuccess) return KS_HIP_ERROR; \
    } while (0)

// ----- device helpers -------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void ks_flag(int32_t *dev_status, int bit) {
    if (dev_status) atomicOr(dev_status, bit);
}

// fp32 -> bf16 bits, round to nearest even (finite inputs; NaN stays NaN)
__device__ __forceinline__ uint32_t ks_f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
// two fp32 -> packed bf16 pair (lo in bits 0-15), round to nearest even: one v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ uint32_t ks_pack_bf2(float lo, float hi) {
    typedef __bf16 ks_bf16x2 __attribute__((ext_vector_type(2)));
    typedef float ks_f32x2 __attribute__((ext_vector_type(2)));
    ks_f32x2 v = {lo, hi};
    ks_bf16x2 b = __builtin_convertvector(v, ks_bf16x2);
    return *(uint32_t *)&b;
}
__device__ __forceinline__ float ks_bf2f(uint32_t b) { return __uint_as_float(b << 16); }

// Reductions and scans of a whole wave (all 64 lanes active) by DPP moves: shifts of 1, 2, 4, 8 lanes inside the rows of 16,
// then the last lane of a row to the next row (0x142) and of the first half to the second (0x143).  A step is one
// vector instruction's latency; the LDS crossbar that __shfl uses costs about 60 cycles a step, which is what the
// small kernels around the sweeps consisted of.  KS_DPP(old, v, ctrl, rows): v of the source lane, `old` where there is none
// or the row is not in the mask.
#define KS_DPP(old, v, ctrl, rows) __builtin_amdgcn_update_dpp(old, v, ctrl, rows, 0xf, false)
#define KS_DPP_F(old, v, ctrl, rows) __int_as_float(KS_DPP(__float_as_int(old), __float_as_int(v), ctrl, rows))
// inclusive scan inside a wave
__device__ __forceinline__ int ks_wave_iscan(int v) {
    v += KS_DPP(0, v, 0x111, 0xf);
    v += KS_DPP(0, v, 0x112, 0xf);
    v += KS_DPP(0, v, 0x114, 0xf);
    v += KS_DPP(0, v, 0x118, 0xf);
    v += KS_DPP(0, v, 0x142, 0xa);
    v += KS_DPP(0, v, 0x143, 0xc);
    return v;
}
__device__ __forceinline__ int ks_wave_max_i(int v) {
    v = max(v, KS_DPP(v, v, 0x111, 0xf));
    v = max(v, KS_DPP(v, v, 0x112, 0xf));
    v = max(v, KS_DPP(v, v, 0x114, 0xf));
    v = max(v, KS_DPP(v, v, 0x118, 0xf));
    v = max(v, KS_DPP(v, v, 0x142, 0xa));
    v = max(v, KS_DPP(v, v, 0x143, 0xc));
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int ks_wave_sum_i(int v) { return __builtin_amdgcn_readlane(ks_wave_iscan(v), 63); }
__device__ __forceinline__ float ks_wave_sum(float v) {
    v += KS_DPP_F(0.f, v, 0x111, 0xf);
    v += KS_DPP_F(0.f, v, 0x112, 0xf);
    v += KS_DPP_F(0.f, v, 0x114, 0xf);
    v += KS_DPP_F(0.f, v, 0x118, 0xf);
    v += KS_DPP_F(0.f, v, 0x142, 0xa);
    v += KS_DPP_F(0.f, v, 0x143, 0xc);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float ks_wave_max(float v) {
    v = fmaxf(v, KS_DPP_F(v, v, 0x111, 0xf));
    v = fmaxf(v, KS_DPP_F(v, v, 0x112, 0xf));
    v = fmaxf(v, KS_DPP_F(v, v, 0x114, 0xf));
    v = fmaxf(v, KS_DPP_F(v, v, 0x118, 0xf));
    v = fmaxf(v, KS_DPP_F(v, v, 0x142, 0xa));
    v = fmaxf(v, KS_DPP_F(v, v, 0x143, 0xc));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// exclusive scan over a block of NT threads (NT multiple of 64, <= 1024); returns the exclusive prefix
// of v, and the block total through *total.  `sh` needs NT/64 + 1 ints of LDS.  Contains barriers.
template <int NT> __device__ __forceinline__ int ks_block_escan(int v, int *sh, int *total) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int inc = ks_wave_iscan(v);
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    const int waves = ks_wave_iscan(lane < NT / 64 ? sh[lane] : 0);
    *total = __builtin_amdgcn_readlane(waves, 63);
    const int r = inc - v + (w ? __builtin_amdgcn_readlane(waves, w - 1) : 0);
    __syncthreads();
    return r;
}
