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

// Eight elements as they are in memory: nothing waits for them before they are used.
typedef __attribute__((ext_vector_type(4))) uint32_t raw_u32x4_t;
template <typename T> struct Raw8 {
    raw_u32x4_t lo, hi;                // (hi: fp32 only)
    __device__ void load(const T* p)
    {
        lo = reinterpret_cast<const raw_u32x4_t*>(p)[0];
        if (sizeof(T) == 4) hi = reinterpret_cast<const raw_u32x4_t*>(p)[1];
    }
    __device__ void store(T* p) const
    {
        reinterpret_cast<raw_u32x4_t*>(p)[0] = lo;
        if (sizeof(T) == 4) reinterpret_cast<raw_u32x4_t*>(p)[1] = hi;
    }
    __device__ void values(float* o) const
    {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            o[i] = __uint_as_float(sizeof(T) == 4 ? (i < 4 ? lo[i & 3] : hi[i & 3]) : i & 1 ? lo[i / 2] & 0xFFFF0000u : lo[i / 2] << 16);
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

// Rotated copies of the queries of rows q_first_row .. Q-1 (copy v of row i turned by qrot0[v] + i): thread qidx
// takes 8 rotary pairs of kPrepHeads heads of a row, which share their (cos, sin), and `vars` of the copies.
// One per (range of copies, sequence, row, group of query heads, group of 8 pairs).  Bound by the
// copies' writes: 9 copies of 4096 rows of 32 heads (0.3 GB) took 97 us with one head per thread and 64-bit
// indices, 79 so (with the chunk's K and V).
constexpr int kPrepHeads = 4;

// as few copies per thread as it takes to give the chip two rounds of threads (every thread reads its queries
// anew); returns the number of threads
inline long query_threads(const Geom& g, const SegList& sl, int q_rows, int* vars)
{
    const long one = (long)g.B * q_rows * ((g.Hq + kPrepHeads - 1) / kPrepHeads) * (g.d / 16);
    int v = sl.n_qvar;
    while (v > 1 && one * ((sl.n_qvar + v - 1) / v) < 2 * 256 * 1024) --v;
    *vars = v;
    return one * ((sl.n_qvar + v - 1) / v);
}

template <typename T>
__device__ inline void rotate_queries(const Geom& g, const SegList& sl, int Q, float qscale, int q_first_row, int vars,
                                      const float2* __restrict__ rope, const T* __restrict__ q, T* __restrict__ Qr, uint32_t qidx)
{
    const int half = g.d / 2, groups = half / 8;
    const uint32_t q_rows = Q - q_first_row, head_groups = (g.Hq + kPrepHeads - 1) / kPrepHeads;
    if (q_rows == 0) return;
    const int e = (int)(qidx % groups) * 8;
    uint32_t r = qidx / groups;
    const int h0 = (int)(r % head_groups) * kPrepHeads;
    r /= head_groups;
    const int i = q_first_row + (int)(r % q_rows);
    r /= q_rows;
    const int b = (int)(r % g.B), v0 = (int)(r / g.B) * vars;
    if (v0 >= sl.n_qvar) return;
    float y0[kPrepHeads][8], y1[kPrepHeads][8];
#pragma unroll
    for (int x = 0; x < kPrepHeads; ++x) {
        const size_t src = (((size_t)b * Q + i) * g.Hq + min(h0 + x, g.Hq - 1)) * g.d;
        Vec8<T>::load(q + src + e, y0[x]);
        Vec8<T>::load(q + src + e + half, y1[x]);
    }
#pragma unroll
    for (int x = 0; x < kPrepHeads; ++x)
#pragma unroll
        for (int j = 0; j < 8; ++j) { y0[x][j] *= qscale; y1[x][j] *= qscale; }
    for (int vq = v0; vq < min(v0 + vars, sl.n_qvar); ++vq) {
        const size_t dst = ((((size_t)vq * g.B + b) * g.Hq + h0) * Q + i) * g.d;
        float2 cs[8];
        const float2* rp = rope + (size_t)(sl.qrot0[vq] + i) * half + e;
#pragma unroll
        for (int j = 0; j < 8; ++j) cs[j] = rp[j];
#pragma unroll
        for (int x = 0; x < kPrepHeads; ++x)
            if (h0 + x < g.Hq) {
                T* to = Qr + dst + (size_t)x * Q * g.d + e;
                rotate8<T>(y0[x], y1[x], cs, to, to + half);
            }
    }
}

}  // namespace ckv
