// Device-side helpers for the gfx950 kernels (wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tka {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// Monotone map float -> uint32: a < b  <=>  ord(a) < ord(b) (for non-NaN; -0 is
// canonicalised to +0 by the caller adding 0.0f).
__device__ __forceinline__ uint32_t ord_from_bits(uint32_t u) {
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ uint32_t bits_from_ord(uint32_t o) {
    return o ^ ((o >> 31) ? 0x80000000u : 0xFFFFFFFFu);
}
// Orders this wave's LDS/global accesses as seen by its own lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// number of set bits of `m` below this lane
__device__ __forceinline__ int mask_rank(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Asks for every 64-byte line of the first BYTES bytes of kernel arguments at once.  A kernel reads its arguments where it needs
// them, and each new line is a trip to memory of its own in a chain of dependent loads.
template <int BYTES>
__device__ __forceinline__ void fetch_args() {
    typedef const __attribute__((address_space(4))) uint32_t* ArgPtr;
    const ArgPtr p = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t v[(BYTES + 63) / 64];
#pragma unroll
    for (int i = 0; i < (BYTES + 63) / 64; ++i) v[i] = p[16 * i];
#pragma unroll
    for (int i = 0; i < (BYTES + 63) / 64; ++i) asm volatile("" ::"s"(v[i]));
}

template <typename T>
__device__ __forceinline__ T wave_xor(T v, int mask) {
    return __shfl_xor(v, mask, 64);
}

// Wave-wide scans and reductions in the vector unit (DPP row shifts and row broadcasts): six instructions, where the
// shuffle form is a chain of six trips through LDS.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f32(float old, float v) {
    return __uint_as_float(dpp_u32<CTRL, ROWS>(__float_as_uint(old), __float_as_uint(v)));
}
// inclusive prefix sum over the 16 lanes of a row
__device__ __forceinline__ uint32_t row_scan_add(uint32_t v) {
    v += dpp_u32<0x111, 0xF>(0u, v);      // row_shr:1
    v += dpp_u32<0x112, 0xF>(0u, v);
    v += dpp_u32<0x114, 0xF>(0u, v);
    v += dpp_u32<0x118, 0xF>(0u, v);
    return v;
}
// inclusive prefix sum over the wave
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v) {
    v = row_scan_add(v);
    v += dpp_u32<0x142, 0xA>(0u, v);      // row_bcast:15 into rows 1 and 3
    v += dpp_u32<0x143, 0xC>(0u, v);      // row_bcast:31 into rows 2 and 3
    return v;
}
// largest value of the wave, in every lane
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_f32<0x111, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_f32<0x112, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_f32<0x114, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_f32<0x118, 0xF>(-INFINITY, v));
    v = fmaxf(v, dpp_f32<0x142, 0xA>(-INFINITY, v));
    v = fmaxf(v, dpp_f32<0x143, 0xC>(-INFINITY, v));
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}
__device__ __forceinline__ float wave_min(float v) { return -wave_max(-v); }
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    uint32_t t;
    t = dpp_u32<0x111, 0xF>(0u, v); v = t > v ? t : v;
    t = dpp_u32<0x112, 0xF>(0u, v); v = t > v ? t : v;
    t = dpp_u32<0x114, 0xF>(0u, v); v = t > v ? t : v;
    t = dpp_u32<0x118, 0xF>(0u, v); v = t > v ? t : v;
    t = dpp_u32<0x142, 0xA>(0u, v); v = t > v ? t : v;
    t = dpp_u32<0x143, 0xC>(0u, v); v = t > v ? t : v;
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// v of this lane + v of lane ^ 16, and the same for lane ^ 32 (register swaps, no trip through LDS)
__device__ __forceinline__ float add_lanes_16(float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_lanes_32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Barrier for what a workgroup exchanges through LDS alone.  (__syncthreads() also waits for every load from memory: the first key
// tile a scan asks for ahead of its thresholds arrived before the second was asked for: 128k tokens 73.9 us per call, now 73.0.)
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum or maximum over groups of LPR neighbouring lanes (4 .. 64, a power of two), in all lanes of the group: a butterfly over
// lane ^ 1, ^ 2, ^ 4, ... in the vector unit.  (Where the lanes of a quad, or of half a row, already agree, the mirrored
// lane holds what the exchanged lane does.)
struct AddOp { static __device__ __forceinline__ float f(float a, float b) { return a + b; } };
struct MaxOp { static __device__ __forceinline__ float f(float a, float b) { return fmaxf(a, b); } };
template <class Op, int LPR>
__device__ __forceinline__ float group_reduce(float v) {
    static_assert(LPR >= 4 && LPR <= 64, "groups of 4 to 64 lanes");
    v = Op::f(v, dpp_f32<0xB1, 0xF>(0.f, v));                  // quad_perm 1,0,3,2
    v = Op::f(v, dpp_f32<0x4E, 0xF>(0.f, v));                  // quad_perm 2,3,0,1
    if (LPR >= 8) v = Op::f(v, dpp_f32<0x141, 0xF>(0.f, v));   // row_half_mirror
    if (LPR >= 16) v = Op::f(v, dpp_f32<0x140, 0xF>(0.f, v));  // row_mirror
    if (LPR >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    if (LPR >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

// widen the 16 bytes a lane loaded into fp32 values
template <int DT> struct Elem;
template <> struct Elem<0> {  // fp32
    static constexpr int kBytes = 4, kPerLoad = 4;
    static __device__ __forceinline__ void widen(const u32x4& r, float* f) {
        f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
        f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
    }
};
template <> struct Elem<1> {  // fp16
    static constexpr int kBytes = 2, kPerLoad = 8;
    static __device__ __forceinline__ void widen(const u32x4& r, float* f) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            union { uint32_t u; _Float16 h[2]; } cv;
            cv.u = w[i];
            f[2 * i] = (float)cv.h[0];
            f[2 * i + 1] = (float)cv.h[1];
        }
    }
};
template <> struct Elem<2> {  // bf16
    static constexpr int kBytes = 2, kPerLoad = 8;
    static __device__ __forceinline__ void widen(const u32x4& r, float* f) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
};

}  // namespace tka
