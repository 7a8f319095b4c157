// storage.h -- conversions between float32 and the storage types.
#pragma once

#include "lq_internal.h"

namespace lq {

// FP32 -> storage conversions of the loader (round to nearest even), the same
// bits on the host and on the device
__host__ __device__ inline uint16_t f32_to_f16_rne(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const uint32_t sign = (u >> 16) & 0x8000u;
    const uint32_t ex = (u >> 23) & 0xFFu;
    uint32_t man = u & 0x7FFFFFu;
    if (ex == 0xFFu) return (uint16_t)(sign | 0x7C00u | (man ? 0x200u : 0u));
    const int e = (int)ex - 127 + 15;
    if (e >= 31) return (uint16_t)(sign | 0x7C00u);          // overflow -> inf
    if (e <= 0) {                                             // subnormal or zero
        if (e < -10) return (uint16_t)sign;
        man |= 0x800000u;
        const int shift = 14 - e;                             // 1 - e + 13
        uint32_t half = man >> shift;
        const uint32_t rem = man & ((1u << shift) - 1u);
        const uint32_t mid = 1u << (shift - 1);
        if (rem > mid || (rem == mid && (half & 1u))) ++half;
        return (uint16_t)(sign | half);
    }
    uint32_t half = ((uint32_t)e << 10) | (man >> 13);
    const uint32_t rem = man & 0x1FFFu;
    if (rem > 0x1000u || (rem == 0x1000u && (half & 1u))) ++half;   // may carry into inf
    return (uint16_t)(sign | half);
}

__host__ __device__ inline uint16_t f32_to_bf16_rne(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
    const uint32_t lsb = (u >> 16) & 1u;
    return (uint16_t)((u + 0x7FFFu + lsb) >> 16);
}

// a stored value widened exactly
__host__ __device__ inline float stored_to_f32(int storage, uint32_t bits) {
    if (storage == LQ_F32) return __builtin_bit_cast(float, bits);
    if (storage == LQ_BF16) return __builtin_bit_cast(float, bits << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}
// density or coefficient as stored, widened again
__host__ __device__ inline float as_stored(int storage, float x) {
    if (storage == LQ_F32) return x;
    return stored_to_f32(storage, storage == LQ_F16 ? f32_to_f16_rne(x) : f32_to_bf16_rne(x));
}

}  // namespace lq
