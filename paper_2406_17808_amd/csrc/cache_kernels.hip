// Cache maintenance kernels: tables, query/key rotation, the score-dependent part of the
// cascade update (Alg. 2) and the row moves that carry it out.
#include "async_copy.h"
#include "launch.h"
#include "plan_core.h"
#include "row_ops.h"
#include "structure.h"

namespace ckv {

// ------------------------------------------------------------------ tables

// (cos, sin)(p * theta_i), theta_i = base^(-2i/d), evaluated in double so that large
// indices keep full float accuracy.
// rope_t (optional): the same values index-minor, [d/4 groups of two rotary pairs][rows], for readers whose
// lanes hold consecutive indices (the attention kernel's queries): their 16-byte loads then fall into
// a few cache lines per instruction instead of one line per lane.
__global__ void rope_table_kernel(float2* __restrict__ rope, float2* __restrict__ rope_t, int rows, int half, int d, double base)
{
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)rows * half) return;
    const int p = (int)(idx / half), i = (int)(idx % half);
    const double theta = pow(base, -2.0 * (double)i / (double)d);
    double s, c;
    sincos((double)p * theta, &s, &c);
    rope[idx] = make_float2((float)c, (float)s);
    if (rope_t) rope_t[((size_t)(i >> 1) * rows + p) * 2 + (i & 1)] = make_float2((float)c, (float)s);
}

void launch_rope_table(const Geom& g, float base, float2* rope, float2* rope_t, int rows, hipStream_t s)
{
    const int half = g.d / 2;
    const long n = (long)rows * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       rope, rope_t, rows, half, g.d, (double)base);
}

// wrow[k] = beta^k (1 - beta): weight of the query row that has k rows after it in its chunk
// (Alg. 3's coefficient; the EMA of Section 3.1 unrolled over the rows of a chunk).
__global__ void wrow_table_kernel(float* __restrict__ wrow, int n, double beta)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) wrow[k] = (float)(pow(beta, (double)k) * (1.0 - beta));
}

void launch_wrow_table(float beta, float* wrow, int n, hipStream_t s)
{
    hipLaunchKernelGGL(wrow_table_kernel, dim3((n + 255) / 256), dim3(256), 0, s, wrow, n, (double)beta);
}

__global__ void fill_i32_kernel(int32_t* __restrict__ p, size_t n, int32_t v)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

void launch_fill_i32(int32_t* p, size_t n, int32_t value, hipStream_t s)
{
    if (n == 0) return;
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 65535);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks), dim3(256), 0, s, p, n, value);
}

// ------------------------------------------------------------------ initial state

// Scatter a state given in cache order into the physical layout (ring heads at 0) and build
// the rotated key copy.  One thread per (row, rotary pair).
struct FillCounts { int sink; int c[kMaxCascades]; };

template <typename T>
__global__ void load_state_kernel(Geom g, FillCounts fc, int total, T* __restrict__ Kc, T* __restrict__ Kr,
                                  T* __restrict__ Vc, float* __restrict__ mu, int32_t* __restrict__ ids,
                                  const float2* __restrict__ rope,
                                  const T* __restrict__ k_in, const T* __restrict__ v_in,
                                  const float* __restrict__ mu_in, const int32_t* __restrict__ ids_in)
{
    const int half = g.d / 2;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long per_bh = (long)total * half;
    if (idx >= per_bh * g.B * g.Hkv) return;
    const int bh = (int)(idx / per_bh);
    const int r = (int)((idx % per_bh) / half), e = (int)(idx % half);
    // rank r in cache order -> physical slot
    int slot = -1, rr = r;
    if (rr < fc.sink) slot = rr;
    else {
        rr -= fc.sink;
        for (int c = g.N - 1; c >= 0; --c) {
            if (rr < fc.c[c]) { slot = g.base[c] + rr; break; }
            rr -= fc.c[c];
        }
    }
    const size_t src = ((size_t)bh * total + r) * g.d;
    const size_t dst = ((size_t)bh * g.slots + slot) * g.d;
    const float x0 = Elem<T>::load(k_in + src + e), x1 = Elem<T>::load(k_in + src + e + half);
    const float2 cs = rope[(size_t)slot * half + e];
    Elem<T>::store(Kc + dst + e, x0);
    Elem<T>::store(Kc + dst + e + half, x1);
    Elem<T>::store(Kr + dst + e, rot_lo(x0, x1, cs.x, cs.y));
    Elem<T>::store(Kr + dst + e + half, rot_hi(x0, x1, cs.x, cs.y));
    Vc[dst + e] = v_in[src + e];
    Vc[dst + e + half] = v_in[src + e + half];
    if (e == 0) {
        mu[(size_t)bh * g.slots + slot] = mu_in[(size_t)bh * total + r];
        ids[(size_t)bh * g.slots + slot] = ids_in[(size_t)bh * total + r];
    }
}

void launch_load_state(const Geom& g, int dtype, const DevBuffers& b, const void* k, const void* v,
                       const float* mu, const int32_t* ids, const int* counts, int total, hipStream_t s)
{
    if (total == 0) return;
    const long n = (long)g.B * g.Hkv * total * (g.d / 2);
    FillCounts fc;
    fc.sink = counts[0];
    for (int i = 0; i < kMaxCascades; ++i) fc.c[i] = i < g.N ? counts[1 + i] : 0;
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (dtype == CASCADE_F32)
        hipLaunchKernelGGL(load_state_kernel<float>, grid, block, 0, s, g, fc, total, (float*)b.Kc, (float*)b.Kr,
                           (float*)b.Vc, b.mu, b.ids, b.rope, (const float*)k, (const float*)v, mu, ids);
    else
        hipLaunchKernelGGL(load_state_kernel<bf16_t>, grid, block, 0, s, g, fc, total, (bf16_t*)b.Kc, (bf16_t*)b.Kr,
                           (bf16_t*)b.Vc, b.mu, b.ids, b.rope, (const bf16_t*)k, (const bf16_t*)v, mu, ids);
}

// ------------------------------------------------------------------ per-chunk rotation

// For every rotated query copy v: Qr[v][b][h][i] = qscale * R(qrot0[v] + i) q[b][i][h] (the bf16
// MFMA kernels want the softmax scale and log2(e) folded into the queries; everybody else passes
// 1); chunk keys are rotated to their chunk index, chunk values are copied head-major.  A thread takes 8 rotary
// pairs of one row (two 16-byte pieces for bf16), or of a few query heads (rotate_queries).
template <typename T>
__global__ void prep_kernel(Geom g, SegList sl, int Q, float qscale, int vars, const float2* __restrict__ rope,
                            const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                            T* __restrict__ Qr, T* __restrict__ Krc, T* __restrict__ Vch)
{
    const int half = g.d / 2, groups = half / 8;
    // threads [0, n_kv): one per (sequence, token, K or V head, group); then those of rotate_queries.  32-bit
    // numbers: 2^32 threads would move more than 128 GB of K and V three times over.
    const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x, n_kv = (uint32_t)g.B * Q * 2 * g.Hkv * groups;
    if (idx < n_kv) {
        const int e = (int)(idx % groups) * 8;
        uint32_t r = idx / groups;
        const int rr = (int)(r % (2 * g.Hkv));
        r /= 2 * g.Hkv;
        const int i = (int)(r % Q), b = (int)(r / Q);
        const int h = rr % g.Hkv;
        const size_t src = (((size_t)b * Q + i) * g.Hkv + h) * g.d;
        const size_t dst = (((size_t)b * g.Hkv + h) * Q + i) * g.d;
        float x0[8], x1[8];
        if (rr < g.Hkv) {
            Vec8<T>::load(k + src + e, x0);
            Vec8<T>::load(k + src + e + half, x1);
            rotate8<T>(x0, x1, rope + (size_t)i * half + e, Krc + dst + e, Krc + dst + e + half);
        } else {
            Vec8<T>::load(v + src + e, x0);
            Vec8<T>::load(v + src + e + half, x1);
            Vec8<T>::store(Vch + dst + e, x0);
            Vec8<T>::store(Vch + dst + e + half, x1);
        }
        return;
    }
    rotate_queries<T>(g, sl, Q, qscale, 0, vars, rope, q, Qr, idx - n_kv);
}

// head dimensions that are not a multiple of 16: one thread per rotary pair
template <typename T>
__global__ void prep_pair_kernel(Geom g, SegList sl, int Q, float qscale, const float2* __restrict__ rope,
                                 const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                 T* __restrict__ Qr, T* __restrict__ Krc, T* __restrict__ Vch)
{
    const int half = g.d / 2;
    const int rows_per_tok = sl.n_qvar * g.Hq + 2 * g.Hkv;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long total = (long)g.B * Q * rows_per_tok * half;
    if (idx >= total) return;
    const int e = (int)(idx % half);
    long r = idx / half;
    const int row = (int)(r % rows_per_tok);
    r /= rows_per_tok;
    const int i = (int)(r % Q), b = (int)(r / Q);
    if (row < sl.n_qvar * g.Hq) {
        const int vq = row / g.Hq, h = row % g.Hq;
        const size_t src = (((size_t)b * Q + i) * g.Hq + h) * g.d;
        const size_t dst = ((((size_t)vq * g.B + b) * g.Hq + h) * Q + i) * g.d;
        const float x0 = qscale * Elem<T>::load(q + src + e), x1 = qscale * Elem<T>::load(q + src + e + half);
        const float2 cs = rope[(size_t)(sl.qrot0[vq] + i) * half + e];
        Elem<T>::store(Qr + dst + e, rot_lo(x0, x1, cs.x, cs.y));
        Elem<T>::store(Qr + dst + e + half, rot_hi(x0, x1, cs.x, cs.y));
    } else {
        const int rr = row - sl.n_qvar * g.Hq;
        const int h = rr % g.Hkv;
        const size_t src = (((size_t)b * Q + i) * g.Hkv + h) * g.d;
        const size_t dst = (((size_t)b * g.Hkv + h) * Q + i) * g.d;
        if (rr < g.Hkv) {
            const float x0 = Elem<T>::load(k + src + e), x1 = Elem<T>::load(k + src + e + half);
            const float2 cs = rope[(size_t)i * half + e];
            Elem<T>::store(Krc + dst + e, rot_lo(x0, x1, cs.x, cs.y));
            Elem<T>::store(Krc + dst + e + half, rot_hi(x0, x1, cs.x, cs.y));
        } else {
            Vch[dst + e] = v[src + e];
            Vch[dst + e + half] = v[src + e + half];
        }
    }
}

void launch_prep(const Geom& g, int dtype, const DevBuffers& b, const SegList& sl, int Q, float qscale,
                 const void* q, const void* k, const void* v, hipStream_t s)
{
    const dim3 block(256);
    if (g.d % 16 == 0) {
        int vars;
        const long n = (long)g.B * Q * 2 * g.Hkv * (g.d / 16) + query_threads(g, sl, Q, &vars);
        const dim3 grid((unsigned)((n + 255) / 256));
        if (dtype == CASCADE_F32)
            hipLaunchKernelGGL(prep_kernel<float>, grid, block, 0, s, g, sl, Q, qscale, vars, b.rope, (const float*)q, (const float*)k,
                               (const float*)v, (float*)b.Qr, (float*)b.Krc, (float*)b.Vch);
        else
            hipLaunchKernelGGL(prep_kernel<bf16_t>, grid, block, 0, s, g, sl, Q, qscale, vars, b.rope, (const bf16_t*)q, (const bf16_t*)k,
                               (const bf16_t*)v, (bf16_t*)b.Qr, (bf16_t*)b.Krc, (bf16_t*)b.Vch);
        return;
    }
    const long n = (long)g.B * Q * (sl.n_qvar * g.Hq + 2 * g.Hkv) * (g.d / 2);
    const dim3 grid((unsigned)((n + 255) / 256));
    if (dtype == CASCADE_F32)
        hipLaunchKernelGGL(prep_pair_kernel<float>, grid, block, 0, s, g, sl, Q, qscale, b.rope, (const float*)q, (const float*)k,
                           (const float*)v, (float*)b.Qr, (float*)b.Krc, (float*)b.Vch);
    else
        hipLaunchKernelGGL(prep_pair_kernel<bf16_t>, grid, block, 0, s, g, sl, Q, qscale, b.rope, (const bf16_t*)q,
                           (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)b.Qr, (bf16_t*)b.Krc, (bf16_t*)b.Vch);
}

// ------------------------------------------------------------------ homogeneous heads

// Appendix "Head Policy and Head Reduction", homogeneous heads: one score per token for all heads.
// The score kernels have reduced the query heads of every KV head; here the KV heads are reduced
// in turn (max of maxima; mean of means, the groups being equally large) and every KV head gets
// the result.  All KV heads then hold the same tokens in the same slots, so the reduction runs
// slot by slot.  For the cached rows the reduction of the updated scores is the update with the
// reduced increments: before the call the scores of a slot are equal in all heads.
__global__ void share_scores_kernel(Geom g, int n_new, int qstride, float* __restrict__ mu, float* __restrict__ mu_chunk)
{
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long per_b = (long)g.slots + n_new;
    if (idx >= per_b * g.B) return;
    const int b = (int)(idx / per_b), j = (int)(idx % per_b);
    float* p = j < g.slots ? mu + (size_t)b * g.Hkv * g.slots + j : mu_chunk + (size_t)b * g.Hkv * qstride + (j - g.slots);
    const size_t stride = j < g.slots ? (size_t)g.slots : (size_t)qstride;
    float r = p[0];
    for (int h = 1; h < g.Hkv; ++h) r = g.head_reduce == CASCADE_REDUCE_MAX ? fmaxf(r, p[h * stride]) : r + p[h * stride];
    if (g.head_reduce == CASCADE_REDUCE_MEAN) r /= (float)g.Hkv;
    for (int h = 0; h < g.Hkv; ++h) p[h * stride] = r;
}

void launch_share_scores(const Geom& g, const DevBuffers& b, int n_new, int max_chunk, hipStream_t s)
{
    const long n = ((long)g.slots + n_new) * g.B;
    hipLaunchKernelGGL(share_scores_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, n_new, max_chunk, b.mu, b.mu_chunk);
}

// ------------------------------------------------------------------ cascade update: who ends up where

// One workgroup per (sequence, KV head).  For every cascade in turn:
//   phase 1  the winner of every segment (see plan_core.h);
//   phase 2  every push passes the item it evicts on to the next cascade.
// winners[c][0] is the segment of the item that was newest before the update, winners[c][1+j]
// that of the j-th slot opened.
__global__ void plan_kernel(Geom g, UpdatePlan pl, int qstride, const float* __restrict__ mu,
                            const float* __restrict__ mu_chunk, int32_t* __restrict__ offers,
                            int32_t* __restrict__ winners, int32_t* __restrict__ swaps)
{
    const int bh = blockIdx.x;
    const float* mub = mu + (size_t)bh * g.slots;
    const float* muc = mu_chunk + (size_t)bh * qstride;
    int32_t* off_in = offers + (size_t)bh * 2 * qstride;
    int32_t* off_out = off_in + qstride;
    for (int c = 0; c < pl.N; ++c) {
        const CascStep cs = pl.c[c];
        if (cs.M == 0) break;
        int32_t* W = winners + ((size_t)bh * pl.N + c) * (qstride + 1);
        const int nseg = cs.J + cs.pre;
        int my_swaps = 0;
        for (int sidx = threadIdx.x; sidx < nseg; sidx += blockDim.x) {
            const int j = sidx - cs.pre;
            int sw;
            W[1 + j] = segment_winner(cs, c, j, g.slots, pl.n_to_sink, g.token_selection, off_in, mub, muc, &sw);
            my_swaps += sw;
        }
        if (my_swaps) atomicAdd(&swaps[bh * pl.N + c], my_swaps);
        __syncthreads();
        for (int i = threadIdx.x; i < cs.P; i += blockDim.x) off_out[i] = evicted_ref(cs, i, W);
        __syncthreads();
        int32_t* tmp = off_in; off_in = off_out; off_out = tmp;
    }
}

void launch_plan(const Geom& g, const DevBuffers& b, const UpdatePlan& pl, int max_chunk, hipStream_t s)
{
    const int threads = pl.Q >= 1024 ? 1024 : (pl.Q >= 256 ? 256 : 64);
    hipLaunchKernelGGL(plan_kernel, dim3(g.B * g.Hkv), dim3(threads), 0, s, g, pl, max_chunk, b.mu, b.mu_chunk,
                       b.offers, b.winners, b.swaps);
}

// ------------------------------------------------------------------ cascade update: row moves

// Final content of cascade c (c = -1: sinks).  Entry e < E names a ring position that was
// written during the update and the ref that ends up in it; one extra entry covers the item
// that was newest before the update if a competing offer replaced it.  A destination row is
// rebuilt from the un-rotated source key, re-rotated to the destination slot index.
// `lanes` threads cooperate on a row; each handles rotary pairs e, e + lanes, ...
template <typename T>
__global__ void move_kernel(Geom g, UpdatePlan pl, int c, int E, int extra, int qstride,
                            const float2* __restrict__ rope, const int32_t* __restrict__ winners,
                            T* __restrict__ Kc, T* __restrict__ Kr, T* __restrict__ Vc,
                            float* __restrict__ mu, int32_t* __restrict__ ids,
                            const float* __restrict__ mu_chunk,
                            const T* __restrict__ k_in, const T* __restrict__ v_in,
                            long tok_stride, long batch_stride, int lanes)
{
    const int bh = blockIdx.y;
    const int b = bh / g.Hkv, h = bh % g.Hkv;
    const int rows_per_block = blockDim.x / lanes;
    const int e = blockIdx.x * rows_per_block + threadIdx.x / lanes;
    const int lane = threadIdx.x % lanes;
    if (e >= E + extra) return;
    int dst, ref;
    if (c < 0) {
        dst = pl.sink_fill0 + e;
        ref = g.slots + e;
    } else {
        const int32_t* W = winners + ((size_t)bh * pl.N + c) * (qstride + 1);
        if (!final_entry(pl.c[c], e, E, W, &dst, &ref)) return;
    }
    const int half = g.d / 2;
    const size_t drow = ((size_t)bh * g.slots + dst) * g.d;
    const T *ks, *vs;
    float score;
    int id;
    if (ref < g.slots) {
        const size_t srow = ((size_t)bh * g.slots + ref) * g.d;
        ks = Kc + srow;
        vs = Vc + srow;
        score = mu[(size_t)bh * g.slots + ref];
        id = ids[(size_t)bh * g.slots + ref];
    } else {
        const int i = ref - g.slots;
        const size_t srow = (size_t)b * batch_stride + (size_t)i * tok_stride + (size_t)h * g.d;
        ks = k_in + srow;
        vs = v_in + srow;
        score = mu_chunk[(size_t)bh * qstride + i];
        id = pl.id0 + i;
    }
    for (int p = lane; p < half; p += lanes) {
        const float x0 = Elem<T>::load(ks + p), x1 = Elem<T>::load(ks + p + half);
        const float2 cs2 = rope[(size_t)dst * half + p];
        Elem<T>::store(Kc + drow + p, x0);
        Elem<T>::store(Kc + drow + p + half, x1);
        Elem<T>::store(Kr + drow + p, rot_lo(x0, x1, cs2.x, cs2.y));
        Elem<T>::store(Kr + drow + p + half, rot_hi(x0, x1, cs2.x, cs2.y));
        Vc[drow + p] = vs[p];
        Vc[drow + p + half] = vs[p + half];
    }
    if (lane == 0) {
        mu[(size_t)bh * g.slots + dst] = score;
        ids[(size_t)bh * g.slots + dst] = id;
    }
}

// The moves of all cascades in two launches.  Every entry (cascade, index) names a destination
// slot and a source; gather_kernel copies the sources that are cache rows (un-rotated key, value,
// score, id: the state before the update) into a staging array, scatter_kernel then writes every
// destination from the staging array or from the chunk's own tokens.  No launch both reads and
// writes the cache, so the order of the cascades does not matter.
struct MoveList {
    int n, total;
    int c[kMaxCascades + 1], first[kMaxCascades + 2], E[kMaxCascades + 1], extra[kMaxCascades + 1];
};

// direct: the plan is direct (plan_is_direct) and nobody has written the winners of the FIRST
// cascade: every token is accepted there (period 1), so a slot it opens takes the offer that opens it
__device__ inline bool move_entry(const Geom& g, const UpdatePlan& pl, const MoveList& ml, int eg, int bh, int qstride,
                                  const int32_t* __restrict__ winners, int* dst, int* ref, bool direct = false)
{
    int i = 0;
    while (i + 1 < ml.n && eg >= ml.first[i + 1]) ++i;
    const int c = ml.c[i], e = eg - ml.first[i];
    if (c < 0) {
        *dst = pl.sink_fill0 + e;
        *ref = g.slots + e;
        return true;
    }
    if (direct && c == 0) {              // J <= cap: entry e is slot j = e; no offer competes in the first cascade
        const CascStep& cs = pl.c[0];
        *dst = cs.base + (cs.wpos0 + e) % cs.cap;
        *ref = offer_ref_direct(pl, 0, e < cs.A ? e : cs.kp0 + (e - cs.A) * cs.pstride, g.slots);
        return true;
    }
    const int32_t* W = winners + ((size_t)bh * pl.N + c) * (qstride + 1);
    return final_entry(pl.c[c], e, ml.E[i], W, dst, ref);
}

// lanes = d/16 threads per row, each moving 8 elements of both halves of the head dimension
template <typename T>
__global__ void gather_kernel(Geom g, UpdatePlan pl, MoveList ml, int qstride, int stage_rows,
                              const int32_t* __restrict__ winners, const T* __restrict__ Kc, const T* __restrict__ Vc,
                              const float* __restrict__ mu, const int32_t* __restrict__ ids,
                              T* __restrict__ stK, T* __restrict__ stV, float* __restrict__ stMu, int32_t* __restrict__ stId)
{
    const int lanes = g.d / 16, half = g.d / 2;
    const int bh = blockIdx.y;
    const int eg = blockIdx.x * (blockDim.x / lanes) + threadIdx.x / lanes;
    const int lane = threadIdx.x % lanes;
    if (eg >= ml.total) return;
    int dst, ref;
    if (!move_entry(g, pl, ml, eg, bh, qstride, winners, &dst, &ref)) return;
    if (ref >= g.slots) return;          // a token of the chunk: read by scatter_kernel
    const size_t srow = ((size_t)bh * g.slots + ref) * g.d, trow = ((size_t)bh * stage_rows + eg) * g.d;
    float x[8];
    Vec8<T>::load(Kc + srow + lane * 8, x);          Vec8<T>::store(stK + trow + lane * 8, x);
    Vec8<T>::load(Kc + srow + half + lane * 8, x);   Vec8<T>::store(stK + trow + half + lane * 8, x);
    Vec8<T>::load(Vc + srow + lane * 8, x);          Vec8<T>::store(stV + trow + lane * 8, x);
    Vec8<T>::load(Vc + srow + half + lane * 8, x);   Vec8<T>::store(stV + trow + half + lane * 8, x);
    if (lane == 0) {
        stMu[(size_t)bh * stage_rows + eg] = mu[(size_t)bh * g.slots + ref];
        stId[(size_t)bh * stage_rows + eg] = ids[(size_t)bh * g.slots + ref];
    }
}

template <typename T>
__global__ void scatter_kernel(Geom g, UpdatePlan pl, MoveList ml, int qstride, int stage_rows,
                               const float2* __restrict__ rope, const int32_t* __restrict__ winners,
                               const T* __restrict__ stK, const T* __restrict__ stV, const float* __restrict__ stMu,
                               const int32_t* __restrict__ stId, const float* __restrict__ mu_chunk,
                               const T* __restrict__ k_in, const T* __restrict__ v_in, long tok_stride, long batch_stride,
                               T* __restrict__ Kc, T* __restrict__ Kr, T* __restrict__ Vc, float* __restrict__ mu,
                               int32_t* __restrict__ ids, bool direct)
{
    const int lanes = g.d / 16, half = g.d / 2;
    const int bh = blockIdx.y;
    const int b = bh / g.Hkv, h = bh % g.Hkv;
    const int eg = blockIdx.x * (blockDim.x / lanes) + threadIdx.x / lanes;
    const int lane = threadIdx.x % lanes;
    if (eg >= ml.total) return;
    int dst, ref;
    if (!move_entry(g, pl, ml, eg, bh, qstride, winners, &dst, &ref, direct)) return;
    const T *ks, *vs;
    float score;
    int id;
    if (ref < g.slots) {
        const size_t trow = ((size_t)bh * stage_rows + eg) * g.d;
        ks = stK + trow;
        vs = stV + trow;
        score = stMu[(size_t)bh * stage_rows + eg];
        id = stId[(size_t)bh * stage_rows + eg];
    } else {
        const int i = ref - g.slots;
        const size_t srow = (size_t)b * batch_stride + (size_t)i * tok_stride + (size_t)h * g.d;
        ks = k_in + srow;
        vs = v_in + srow;
        score = mu_chunk[(size_t)bh * qstride + i];
        id = pl.id0 + i;
    }
    const size_t drow = ((size_t)bh * g.slots + dst) * g.d;
    const int e = lane * 8;
    float x0[8], x1[8];
    Vec8<T>::load(ks + e, x0);
    Vec8<T>::load(ks + half + e, x1);
    Vec8<T>::store(Kc + drow + e, x0);
    Vec8<T>::store(Kc + drow + half + e, x1);
    rotate8<T>(x0, x1, rope + (size_t)dst * half + e, Kr + drow + e, Kr + drow + half + e);
    Vec8<T>::load(vs + e, x0);
    Vec8<T>::load(vs + half + e, x1);
    Vec8<T>::store(Vc + drow + e, x0);
    Vec8<T>::store(Vc + drow + half + e, x1);
    if (lane == 0) {
        mu[(size_t)bh * g.slots + dst] = score;
        ids[(size_t)bh * g.slots + dst] = id;
    }
}

// The winner of segment j of cascade c (j = -1: the newest item's), under plan_is_direct, decided by the `lanes` threads of a
// group together: the same first-maximum rule as segment_winner (a later offer replaces the holder only on a strictly higher
// score), with the scores of `lanes` offers loaded at a time instead of one after the other.  Groups lie inside a wave; all
// lanes of the wave call it (c < 0: nothing to decide).  Returns the ref, *dst the slot, *swaps the replacements.
__device__ inline int direct_winner(const Geom& g, const UpdatePlan& pl, int c, int j, int lanes, int lane, const float* __restrict__ mub,
                                    const float* __restrict__ muc, int* dst, int* swaps)
{
    const int lead = (threadIdx.x & 63) - lane;              // first lane of this group inside the wave
    int ref = 0, kb = 0, ke = 0, sw = 0;
    float bs = 0.f;
    if (c >= 0) {
        const CascStep& cs = pl.c[c];
        if (j < 0) {
            *dst = ref = cs.base + cs.newest0;
        } else {
            *dst = cs.base + ring_position(cs, j);
            kb = segment_first_offer(cs, j);
            ref = offer_ref_direct(pl, c, kb, g.slots);
            ++kb;
        }
        ke = g.token_selection ? segment_first_offer(cs, j + 1) : kb;
        if (ke > kb) bs = ref_score(ref, g.slots, mub, muc);
    }
    // rounds of `lanes` offers; groups of one wave may need different numbers of rounds
    const int rounds = ke > kb ? (ke - kb + lanes - 1) / lanes : 0;
    int max_rounds = rounds;
    for (int w = lanes; w < 64; w <<= 1) max_rounds = max(max_rounds, __shfl_xor(max_rounds, w, 64));
    for (int r = 0; r < max_rounds; ++r) {
        const int k = kb + r * lanes + lane;
        const bool valid = r < rounds && k < ke;
        int rk = 0;
        float s = -INFINITY;
        if (valid) {
            rk = offer_ref_direct(pl, c, k, g.slots);
            s = ref_score(rk, g.slots, mub, muc);
        }
        // highest score among the holder and the offers before this lane's
        float before = bs;
        for (int x = 0; x < lanes; ++x) {
            const float sx = __shfl(s, lead + x, 64);
            if (x < lane) before = fmaxf(before, sx);
        }
        const bool record = valid && s > before;             // this offer would replace the holder when its turn comes
        const unsigned long long rec = __ballot(record) >> lead & ((1ull << lanes) - 1ull);
        if (rec) {
            const int last = 63 - __builtin_clzll(rec);      // the last replacement of the round holds the slot after it
            ref = __shfl(rk, lead + last, 64);
            bs = __shfl(s, lead + last, 64);
            sw += __builtin_popcountll(rec);
        }
    }
    *swaps = sw;
    return ref;
}

// A direct update in one launch: a workgroup takes whole trees (MoveTrees), a thread group ND slots of them.  It decides who
// ends up in its slots, reads those rows and, when every group of the workgroup has read its own, writes
// them: nobody else reads or writes the slots of these trees, so no row has to be staged in memory.
// Bound by latency (offers, scores, rows, stores, one after the other) where it is small, by memory from 4096 tokens on.  Against
// a launch that decides and stages and one that writes, us with 8 KV heads: 512 tokens 12.7 -> 7.5, 1024 14.9 -> 10.8, 2048 with
// eight cascades 24.9 -> 14.8, 4096 36.3 -> 30.3; fp32, 32 tokens, one head 9.3 -> 6.0.
template <typename T, int ND>
__global__ __launch_bounds__(1024) void move_trees_kernel(Geom g, UpdatePlan pl_arg, MoveTrees mt_arg, int qstride, const float2* __restrict__ rope,
                                                          const float* __restrict__ mu_chunk, const T* __restrict__ k_in, const T* __restrict__ v_in,
                                                          long tok_stride, long batch_stride, T* Kc, T* __restrict__ Kr, T* Vc, float* mu,
                                                          int32_t* ids, int32_t* __restrict__ swaps)
{
    // The plan lies in LDS: one load for all of it, where every look at an argument is a load of its own, most of them one
    // after the other, with cold caches.
    __shared__ UpdatePlan pl;
    __shared__ MoveTrees mt;
    __shared__ int wg_swaps[kMaxCascades];   // replacements counted by this workgroup, per cascade
    const int lanes = g.d / 16, half = g.d / 2, groups = blockDim.x / lanes;
    const int bh = blockIdx.y, b = bh / g.Hkv, h = bh % g.Hkv;
    const int grp = threadIdx.x / lanes, lane = threadIdx.x % lanes;
    for (int i = threadIdx.x; i < (int)(sizeof(UpdatePlan) / 4); i += blockDim.x)
        reinterpret_cast<int*>(&pl)[i] = reinterpret_cast<const int*>(&pl_arg)[i];
    for (int i = threadIdx.x; i < (int)(sizeof(MoveTrees) / 4); i += blockDim.x)
        reinterpret_cast<int*>(&mt)[i] = reinterpret_cast<const int*>(&mt_arg)[i];
    if (threadIdx.x < kMaxCascades) wg_swaps[threadIdx.x] = 0;
    __syncthreads();
    int cls = 0;
    while (cls + 1 < mt.n && (int)blockIdx.x >= mt.first_wg[cls + 1]) ++cls;
    const int root = mt.c[cls], r0 = ((int)blockIdx.x - mt.first_wg[cls]) * mt.per[cls], r1 = min(mt.count[cls], r0 + mt.per[cls]);
    int ref[ND], dst[ND], id[ND];
    float score[ND];
    bool move[ND];
    Raw8<T> k0[ND], k1[ND], v0[ND], v1[ND];
    float2 cs[ND][8];                        // of the destination
#pragma unroll
    for (int n = 0; n < ND; ++n) {
        // this group's slot: the trees' segments cascade by cascade, the roots first
        const int x = n * groups + grp;
        int c = -2, j = 0;
        if (root < 0) {
            if (x < r1 - r0) { c = -1; j = r0 + x; }
        } else {
            int j0 = mt.lo[cls] + r0, j1 = mt.lo[cls] + r1, ahead = 0;
            for (int lc = root;; --lc) {
                if (x >= ahead && x < ahead + j1 - j0) { c = lc; j = j0 + x - ahead; }
                ahead += j1 - j0;
                if (lc == 0) break;
                child_segments(pl, lc, &j0, &j1);
            }
        }
        int sw = 0;
        ref[n] = direct_winner(g, pl, c, j, lanes, lane, mu + (size_t)bh * g.slots, mu_chunk + (size_t)bh * qstride, &dst[n], &sw);
        if (c == -1) { dst[n] = pl.sink_fill0 + j; ref[n] = g.slots + j; }
        if (lane == 0 && sw) atomicAdd(&wg_swaps[c], sw);
        move[n] = c >= -1 && ref[n] != dst[n];
        if (move[n]) {
            const T *ks, *vs;
            if (ref[n] < g.slots) {
                const size_t srow = (size_t)bh * g.slots + ref[n];
                ks = Kc + srow * g.d;
                vs = Vc + srow * g.d;
                score[n] = mu[srow];
                id[n] = ids[srow];
            } else {
                const int i = ref[n] - g.slots;
                const size_t srow = (size_t)b * batch_stride + (size_t)i * tok_stride + (size_t)h * g.d;
                ks = k_in + srow;
                vs = v_in + srow;
                score[n] = mu_chunk[(size_t)bh * qstride + i];
                id[n] = pl.id0 + i;
            }
            k0[n].load(ks + lane * 8);
            k1[n].load(ks + half + lane * 8);
            v0[n].load(vs + lane * 8);
            v1[n].load(vs + half + lane * 8);
#pragma unroll
            for (int i = 0; i < 8; ++i) cs[n][i] = rope[(size_t)dst[n] * half + lane * 8 + i];
        }
    }
    wait_vm_fenced<0>();                     // (a barrier alone need not wait for loads)
    __syncthreads();
#pragma unroll
    for (int n = 0; n < ND; ++n)
        if (move[n]) {
            const size_t drow = ((size_t)bh * g.slots + dst[n]) * g.d;
            const int e = lane * 8;
            k0[n].store(Kc + drow + e);
            k1[n].store(Kc + drow + half + e);
            v0[n].store(Vc + drow + e);
            v1[n].store(Vc + drow + half + e);
            float x0[8], x1[8];
            k0[n].values(x0);
            k1[n].values(x1);
            rotate8<T>(x0, x1, cs[n], Kr + drow + e, Kr + drow + half + e);
            if (lane == 0) {
                mu[(size_t)bh * g.slots + dst[n]] = score[n];
                ids[(size_t)bh * g.slots + dst[n]] = id[n];
            }
        }
    if (threadIdx.x < pl.N && wg_swaps[threadIdx.x]) atomicAdd(&swaps[bh * pl.N + threadIdx.x], wg_swaps[threadIdx.x]);
}

// gather_kernel for updates whose plan is direct (plan_is_direct): the thread group of an entry
// decides its segment itself (the offers are named from the structure alone), leaves the winner
// in `winners` for scatter_kernel, counts the replacements, and stages the winner if it is a cache
// row.  No plan_kernel launch, no cascade-by-cascade dependency.  Only the cascades beyond the
// first have anything to decide or to stage (the first takes the chunk's tokens as they come):
// the launch covers their entries only, n_entries of them.
template <typename T>
__global__ void gather_direct_kernel(Geom g, UpdatePlan pl, MoveList ml, int n_entries, int qstride, int stage_rows,
                                     int32_t* __restrict__ winners, int32_t* __restrict__ swaps,
                                     const float* __restrict__ mu_chunk, const T* __restrict__ Kc, const T* __restrict__ Vc,
                                     const float* __restrict__ mu, const int32_t* __restrict__ ids,
                                     T* __restrict__ stK, T* __restrict__ stV, float* __restrict__ stMu, int32_t* __restrict__ stId)
{
    __shared__ int wg_swaps[kMaxCascades];   // replacements counted by this workgroup, per cascade
    const int lanes = g.d / 16, half = g.d / 2;
    const int bh = blockIdx.y;
    const int eg = blockIdx.x * (blockDim.x / lanes) + threadIdx.x / lanes;
    const int lane = threadIdx.x % lanes;
    if (threadIdx.x < kMaxCascades) wg_swaps[threadIdx.x] = 0;
    __syncthreads();
    int c = -1, j = 0, dst = 0;
    if (eg < n_entries) {                // the entries of the cascades beyond the first come first in the list
        int i = 0;
        while (i + 1 < ml.n && eg >= ml.first[i + 1]) ++i;
        c = ml.c[i];
        {
            // entry e < E is slot j = e of the J <= cap slots opened (final_entry); entry E is the segment of
            // the item that was newest before the update
            const int e = eg - ml.first[i];
            j = e < ml.E[i] ? e : -1;
        }
    }
    int sw;
    const int ref = direct_winner(g, pl, c, j, lanes, lane, mu + (size_t)bh * g.slots, mu_chunk + (size_t)bh * qstride, &dst, &sw);
    if (c >= 0 && lane == 0) {
        winners[((size_t)bh * pl.N + c) * (qstride + 1) + 1 + j] = ref;
        if (sw) atomicAdd(&wg_swaps[c], sw);
    }
    const bool move = c >= 0 && ref < g.slots && ref != dst;   // a cache row that goes somewhere else (chunk tokens are read by scatter_kernel)
    if (move) {
        const size_t srow = ((size_t)bh * g.slots + ref) * g.d, trow = ((size_t)bh * stage_rows + eg) * g.d;
        float x[8];
        Vec8<T>::load(Kc + srow + lane * 8, x);          Vec8<T>::store(stK + trow + lane * 8, x);
        Vec8<T>::load(Kc + srow + half + lane * 8, x);   Vec8<T>::store(stK + trow + half + lane * 8, x);
        Vec8<T>::load(Vc + srow + lane * 8, x);          Vec8<T>::store(stV + trow + lane * 8, x);
        Vec8<T>::load(Vc + srow + half + lane * 8, x);   Vec8<T>::store(stV + trow + half + lane * 8, x);
        if (lane == 0) {
            stMu[(size_t)bh * stage_rows + eg] = mu[(size_t)bh * g.slots + ref];
            stId[(size_t)bh * stage_rows + eg] = ids[(size_t)bh * g.slots + ref];
        }
    }
    __syncthreads();
    if (threadIdx.x < pl.N && wg_swaps[threadIdx.x]) atomicAdd(&swaps[bh * pl.N + threadIdx.x], wg_swaps[threadIdx.x]);
}

template <typename T>
static void moves_two_phase(const Geom& g, const DevBuffers& b, const UpdatePlan& pl, const MoveList& ml, int max_chunk,
                            const void* k, const void* v, int k_token_stride, int k_batch_stride, bool direct, hipStream_t s)
{
    const int lanes = g.d / 16, threads = 256, rows = threads / lanes;
    const dim3 grid((ml.total + rows - 1) / rows, g.B * g.Hkv), block(threads);
    const size_t BH = (size_t)g.B * g.Hkv;
    T* stK = (T*)b.move_stage;
    T* stV = stK + BH * b.move_stage_rows * g.d;
    float* stMu = (float*)(stV + BH * b.move_stage_rows * g.d);
    int32_t* stId = (int32_t*)(stMu + BH * b.move_stage_rows);
    if (direct) {
        int n_entries = ml.total;        // entries before those of the first cascade and of the sinks
        for (int i = 0; i < ml.n; ++i)
            if (ml.c[i] <= 0) { n_entries = ml.first[i]; break; }
        if (n_entries > 0)
            hipLaunchKernelGGL(gather_direct_kernel<T>, dim3((n_entries + rows - 1) / rows, g.B * g.Hkv), block, 0, s, g, pl, ml, n_entries,
                               max_chunk, b.move_stage_rows, b.winners, b.swaps, b.mu_chunk, (const T*)b.Kc, (const T*)b.Vc, b.mu, b.ids,
                               stK, stV, stMu, stId);
    } else
        hipLaunchKernelGGL(gather_kernel<T>, grid, block, 0, s, g, pl, ml, max_chunk, b.move_stage_rows, b.winners,
                           (const T*)b.Kc, (const T*)b.Vc, b.mu, b.ids, stK, stV, stMu, stId);
    hipLaunchKernelGGL(scatter_kernel<T>, grid, block, 0, s, g, pl, ml, max_chunk, b.move_stage_rows, b.rope, b.winners,
                       (const T*)stK, (const T*)stV, stMu, stId, b.mu_chunk, (const T*)k, (const T*)v,
                       (long)k_token_stride, (long)k_batch_stride, (T*)b.Kc, (T*)b.Kr, (T*)b.Vc, b.mu, b.ids, direct);
}

// Head dimensions that are not a multiple of 16 take one launch per cascade: destinations of
// cascade c take sources from earlier cascades or from the chunk only (items never move
// backwards), so writing the last cascade first keeps every source intact until it has been read.
bool update_is_direct(const Geom& g, const DevBuffers& b, const UpdatePlan& pl)
{
    if (!(g.d % 16 == 0 && b.move_stage) || 64 % (g.d / 16) != 0 || b.opt_update_staged || !plan_is_direct(pl)) return false;   // (thread groups inside a wave)
    int total = pl.n_to_sink;
    for (int c = 0; c < pl.N; ++c) {
        if (pl.c[c].M == 0) continue;
        int extra;
        total += final_entries(pl.c[c], &extra);
        total += extra;
    }
    return total <= b.move_stage_rows;
}

// A direct update whose trees fit workgroups: as few threads as hold the largest tree.  The trees of N cascades with the default
// periods have up to 2^N - 1 slots; false where a tree has more than 1024 threads hold, d / 16 of them for two slots (from ten
// cascades on at d = 64, nine at 128, eight at 256, fewer with long periods): such updates go through the staging array.
template <typename T>
static bool moves_of_trees(const Geom& g, const DevBuffers& b, const UpdatePlan& pl, int max_chunk, const void* k, const void* v, int k_token_stride,
                           int k_batch_stride, hipStream_t s)
{
    const int lanes = g.d / 16;
    MoveTrees mt;
    for (int x = 0; x < 4; ++x) {
        const int threads = x < 2 ? 256 << x : 1024, nodes = x < 3 ? 1 : 2;
        plan_trees(pl, threads / lanes * nodes, mt);
        if (mt.wgs == 0) continue;
        const dim3 grid(mt.wgs, g.B * g.Hkv), block(threads);
        if (nodes == 1)
            hipLaunchKernelGGL((move_trees_kernel<T, 1>), grid, block, 0, s, g, pl, mt, max_chunk, b.rope, b.mu_chunk, (const T*)k, (const T*)v,
                               (long)k_token_stride, (long)k_batch_stride, (T*)b.Kc, (T*)b.Kr, (T*)b.Vc, b.mu, b.ids, b.swaps);
        else
            hipLaunchKernelGGL((move_trees_kernel<T, 2>), grid, block, 0, s, g, pl, mt, max_chunk, b.rope, b.mu_chunk, (const T*)k, (const T*)v,
                               (long)k_token_stride, (long)k_batch_stride, (T*)b.Kc, (T*)b.Kr, (T*)b.Vc, b.mu, b.ids, b.swaps);
        return true;
    }
    return false;
}

// `direct`: no plan_kernel has run; the launches decide the segments themselves (update_is_direct)
void launch_moves(const Geom& g, int dtype, const DevBuffers& b, const UpdatePlan& pl, int max_chunk,
                  const void* k, const void* v, int k_token_stride, int k_batch_stride, bool direct, hipStream_t s)
{
    if (direct &&
        (dtype == CASCADE_F32 ? moves_of_trees<float>(g, b, pl, max_chunk, k, v, k_token_stride, k_batch_stride, s)
                              : moves_of_trees<bf16_t>(g, b, pl, max_chunk, k, v, k_token_stride, k_batch_stride, s)))
        return;
    if (g.d % 16 == 0 && b.move_stage) {
        MoveList ml;
        ml.n = 0;
        ml.total = 0;
        for (int c = pl.N - 1; c >= -1; --c) {
            int E, extra = 0;
            if (c < 0) {
                E = pl.n_to_sink;
            } else {
                if (pl.c[c].M == 0) continue;
                E = final_entries(pl.c[c], &extra);
            }
            if (E + extra == 0) continue;
            ml.c[ml.n] = c; ml.first[ml.n] = ml.total; ml.E[ml.n] = E; ml.extra[ml.n] = extra;
            ml.total += E + extra;
            ++ml.n;
        }
        ml.first[ml.n] = ml.total;
        if (ml.total == 0) return;
        if (ml.total <= b.move_stage_rows) {
            if (dtype == CASCADE_F32) moves_two_phase<float>(g, b, pl, ml, max_chunk, k, v, k_token_stride, k_batch_stride, direct, s);
            else moves_two_phase<bf16_t>(g, b, pl, ml, max_chunk, k, v, k_token_stride, k_batch_stride, direct, s);
            return;
        }
    }
    const int lanes = 32, threads = 256, rows = threads / lanes;
    for (int c = pl.N - 1; c >= -1; --c) {
        int E, extra = 0;
        if (c < 0) {
            E = pl.n_to_sink;
        } else {
            if (pl.c[c].M == 0) continue;
            E = final_entries(pl.c[c], &extra);
        }
        if (E + extra == 0) continue;
        const dim3 grid((E + extra + rows - 1) / rows, g.B * g.Hkv), block(threads);
        if (dtype == CASCADE_F32)
            hipLaunchKernelGGL(move_kernel<float>, grid, block, 0, s, g, pl, c, E, extra, max_chunk, b.rope, b.winners,
                               (float*)b.Kc, (float*)b.Kr, (float*)b.Vc, b.mu, b.ids, b.mu_chunk,
                               (const float*)k, (const float*)v, (long)k_token_stride, (long)k_batch_stride, lanes);
        else
            hipLaunchKernelGGL(move_kernel<bf16_t>, grid, block, 0, s, g, pl, c, E, extra, max_chunk, b.rope, b.winners,
                               (bf16_t*)b.Kc, (bf16_t*)b.Kr, (bf16_t*)b.Vc, b.mu, b.ids, b.mu_chunk,
                               (const bf16_t*)k, (const bf16_t*)v, (long)k_token_stride, (long)k_batch_stride, lanes);
    }
}

}  // namespace ckv
