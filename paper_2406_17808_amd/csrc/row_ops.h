// Device helpers that move cache rows: eight elements at a time, and the rotation of eight rotary pairs.
#pragma once

#include "internal.h"

namespace ckv {

template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> {
    __device__ static void load(const bf16_t* p, float* o)
    {
        const uint4 u = *reinterpret_cast<const uint4*>(p);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[2 * i] = __uint_as_float(w[i] << 16); o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u); }
    }
    __device__ static void store(bf16_t* p, const float* v)
    {
        uint4 u;
        u.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
        u.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
        u.z = (uint32_t)f32_to_bf16(v[4]) | ((uint32_t)f32_to_bf16(v[5]) << 16);
        u.w = (uint32_t)f32_to_bf16(v[6]) | ((uint32_t)f32_to_bf16(v[7]) << 16);
        *reinterpret_cast<uint4*>(p) = u;
    }
};
template <> struct Vec8<float> {
    __device__ static void load(const float* p, float* o)
    {
        const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    }
    __device__ static void store(float* p, const float* v)
    {
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
};

template <typename T>
__device__ inline void rotate8(const float* x0, const float* x1, const float2* __restrict__ cs, T* d0, T* d1)
{
    float y0[8], y1[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float2 c = cs[i];
        y0[i] = rot_lo(x0[i], x1[i], c.x, c.y);
        y1[i] = rot_hi(x0[i], x1[i], c.x, c.y);
    }
    Vec8<T>::store(d0, y0);
    Vec8<T>::store(d1, y1);
}

}  // namespace ckv
