// The quantizer's element rules with compile-time formats, shared by the quantize kernels: block scale,
// rank of a magnitude through the format's table, source unpacking.
#pragma once

#include <cstdint>
#include <hip/hip_runtime.h>

#include "curvefp_internal.hpp"

namespace curvefp {

template <class F>
__device__ __forceinline__ int block_scale(uint32_t amax, uint32_t lmax_mant) {
    // an all-zero block (every integer a satisfies 0 <= 2^a fl32(L_max)) and a subnormal maximum
    // both take the bottom of the scale range
    const int ef = (int)(amax >> 23);
    if (ef == 0) return -127;
    const int a = ef - 127 - F::OHI + (((amax & 0x7FFFFFu) > lmax_mant) ? 1 : 0);
    return min(max(a, -127), 127);
}

// rank of y whose fp32 bit pattern is yb (already scaled), table in LDS
template <class F>
__device__ __forceinline__ uint32_t rank_lookup(int32_t yb, const uint32_t* lut) {
    int32_t idx = (yb >> 16) - ((127 + F::OZ) << 7);
    if (idx < 0) return 0;
    idx = min(idx, F::QLUT_SIZE - 1);
    const uint32_t e = lut[idx];
    return (e >> 16) + ((((uint32_t)yb & 0xFFFFu) > (e & 0xFFFFu)) ? 1u : 0u);
}

// the same for a yb whose low 16 bits are zero, with the one-byte table
template <class F>
__device__ __forceinline__ uint32_t rank_lookup(int32_t yb, const uint8_t* lut) {
    int32_t idx = (yb >> 16) - ((127 + F::OZ) << 7);
    if (idx < 0) return 0;
    return lut[min(idx, F::QLUT_SIZE - 1)];
}

// fast path: a >= A_FAST_MIN, where subnormal or zero inputs can only reach rank 0
template <class F, class T>
__device__ __forceinline__ uint32_t rank_fast(uint32_t mag, int a, const T* lut) {
    return rank_lookup<F>((int32_t)mag - (a << 23), lut);
}

// exact path for blocks with tiny scales: normalize subnormal inputs first
template <class F, class T>
__device__ __forceinline__ uint32_t rank_exact(uint32_t mag, int a, const T* lut) {
    if (mag == 0) return 0;
    int32_t yb;
    if ((mag >> 23) == 0) {
        const int p = 31 - __clz(mag);              // position of the leading one, 0..22
        const uint32_t mn = mag << (23 - p);
        yb = (int32_t)(((uint32_t)(p - 22 - a) << 23) | (mn & 0x7FFFFFu));
    } else {
        yb = (int32_t)mag - (a << 23);
    }
    return rank_lookup<F>(yb, lut);
}

template <class F, class T>
__device__ __forceinline__ void ranks_of(const uint32_t* mag, int n, int a, const T* lut, uint32_t* r) {
    if (a == -128) {
        for (int i = 0; i < n; i++) r[i] = 0;
    } else if (a >= F::A_FAST_MIN) {
        for (int i = 0; i < n; i++) r[i] = rank_fast<F>(mag[i], a, lut);
    } else {
        for (int i = 0; i < n; i++) r[i] = rank_exact<F>(mag[i], a, lut);
    }
}

template <class F>
__device__ __forceinline__ int scale_of(uint32_t amax, uint32_t lmax_mant) {
    return (amax >= 0x7F800000u) ? -128 : block_scale<F>(amax, lmax_mant);
}

// unpack 8 consecutive source elements into magnitude bits (as fp32) and sign bits
template <bool BF16>
__device__ __forceinline__ void unpack8(const uint4* v, uint32_t* mag, uint32_t* sgn) {
    if (BF16) {
        const uint32_t w[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            mag[2 * i] = (w[i] << 16) & 0x7FFF0000u;
            mag[2 * i + 1] = w[i] & 0x7FFF0000u;
            sgn[2 * i] = (w[i] >> 15) & 1u;
            sgn[2 * i + 1] = w[i] >> 31;
        }
    } else {
        const uint32_t w[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
        for (int i = 0; i < 8; i++) {
            mag[i] = w[i] & 0x7FFFFFFFu;
            sgn[i] = w[i] >> 31;
        }
    }
}

}  // namespace curvefp
