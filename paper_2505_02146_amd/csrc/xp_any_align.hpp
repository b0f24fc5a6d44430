// Loads of 16-byte chunks that start at any element, masks for their parts, and the 16x16 matrix instructions: what the
// kernels for operands of any alignment share.
#pragma once

#include <hip/hip_runtime.h>

namespace xp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef unsigned int u32x4_dw __attribute__((ext_vector_type(4), aligned(4)));

template <bool INT8> struct Kind;
template <> struct Kind<false> {
    static constexpr int ESZ = 2;
    typedef f32x4 acc_t;
    typedef float out_t;
    typedef unsigned short elem;
    static __device__ __forceinline__ acc_t mma(u32x4 a, u32x4 b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Kind<true> {
    static constexpr int ESZ = 1;
    typedef i32x4 acc_t;
    typedef int out_t;
    typedef unsigned char elem;
    static __device__ __forceinline__ acc_t mma(u32x4 a, u32x4 b, acc_t c)
    {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
    }
};

__device__ __forceinline__ u32x4 load16(const char *p) { return *(const u32x4_any *)p; }

// the same for data that is used once
__device__ __forceinline__ u32x4 load16_stream(const char *p) { return __builtin_nontemporal_load((const u32x4_any *)p); }

// The chunk at base + at, of which only bytes in [first, last) are read, `last - first` being 16 or more: where it sticks
// out, the nearest 16 bytes inside are loaded and moved to their places (zeros beside them).
__device__ __forceinline__ u32x4 load16_within(const char *base, long long at, long long first, long long last)
{
    const long long from = at < first ? first : (at + 16 > last ? last - 16 : at);
    u32x4 v = load16(base + from);
    const int by = (int)(at - from);                             // -15 .. 15 where the chunk holds anything
    if (__builtin_amdgcn_ballot_w64(by != 0) != 0) {
        unsigned long long lo = ((unsigned long long)v[1] << 32) | v[0], hi = ((unsigned long long)v[3] << 32) | v[2];
        const int n = 8 * (by < 0 ? -by : by);
        if (by > 0) {
            lo = n >= 64 ? hi >> (n & 63) : (lo >> n) | (hi << 1 << (63 - n));
            hi = n >= 64 ? 0ull : hi >> n;
        } else if (by < 0) {
            hi = n >= 64 ? lo << (n & 63) : (hi << n) | (lo >> 1 >> (63 - n));
            lo = n >= 64 ? 0ull : lo << n;
        }
        v = u32x4{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
    }
    return v;
}

// bit i set: element i of the chunk counts
template <int ESZ> __device__ __forceinline__ u32x4 keep(u32x4 v, unsigned bits)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        unsigned m;
        if constexpr (ESZ == 2) {
            m = ((unsigned)__builtin_amdgcn_sbfe((int)bits, 2 * d, 1) & 0xffffu) | ((unsigned)__builtin_amdgcn_sbfe((int)bits, 2 * d + 1, 1) << 16);
        } else {
            const unsigned n = (bits >> (4 * d)) & 15u;
            m = ((n * 0x00204081u) & 0x01010101u) * 0xffu;
        }
        v[d] &= m;
    }
    return v;
}

}  // namespace xp
