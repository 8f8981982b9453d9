// Chunk attention and score sums in fp32 on the matrix cores (head dimension 64 or 128): the fp32
// configuration.  The arithmetic is fp32 throughout; v_mfma_f32_16x16x4_f32 takes fp32 operands.
//
// v_mfma_f32_16x16x4_f32, D[m][n] += sum_k A[m][k] B[k][n]: lane l holds A[l%16][l/16] and
// B[l/16][l%16]; D: column l%16, rows 4*(l/16) .. +3.  Which element of the head dimension a
// contraction index means is free as long as A and B agree: lane group c = l/16 takes elements
// c*D/4 + step, so a lane reads D/4 contiguous floats of its row.
#include <type_traits>

#include "launch.h"

namespace ckv {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr float kF32Log2e = 1.4426950408889634f;
constexpr int kF32Keys = 16;       // keys per tile

template <int D> __device__ inline void load_quarter(const float* __restrict__ row, int c, float (&x)[D / 4])
{
#pragma unroll
    for (int i = 0; i < D / 4; i += 4) *reinterpret_cast<f32x4_t*>(&x[i]) = *reinterpret_cast<const f32x4_t*>(row + c * (D / 4) + i);
}

template <int D> __device__ inline f32x4_t product(const float (&a)[D / 4], const float (&b)[D / 4])
{
    // two accumulators: a chain of dependent MFMAs is half as long
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int i = 0; i < D / 4; i += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i + 1], b[i + 1], s1, 0, 0, 0);
    }
    return s0 + s1;
}

__device__ inline float max_of_groups(float x)   // over lanes l, l^16, l^32, l^48
{
    x = fmaxf(x, __shfl_xor(x, 16, 64));
    return fmaxf(x, __shfl_xor(x, 32, 64));
}

// O^T += V^T P^T for the keys of one tile that a row sees (those before `end`), product by product.
template <int D>
__device__ inline void add_visible(const float* __restrict__ vbase, int k0, int end, int n, int c, const float (&p)[4], f32x4_t (&o)[D / 16])
{
    for (int x = 0; x < kF32Keys; ++x) {
        const int j = x & 3;
        const float px = __shfl(j == 0 ? p[0] : j == 1 ? p[1] : j == 2 ? p[2] : p[3], (x >> 2) * 16 + n, 64);   // key x of this lane's row
        if (k0 + x >= end) continue;
        const f32x4_t* v = reinterpret_cast<const f32x4_t*>(vbase + (size_t)(k0 + x) * D + 4 * c);
#pragma unroll
        for (int db = 0; db < D / 16; ++db) o[db] += v[4 * db] * px;
    }
}

// ------------------------------------------------------------------ attention
//
// A workgroup owns 16 (head, token) rows of one KV head; its eight waves take the 16-key tiles in turn,
// each with its own running maximum, and are combined at the end: small launches, which is what this
// configuration is for, are bound by the latency of one wave's tiles, so the keys are spread over waves.
// S^T = K Q^T leaves query l%16 and keys 4*(l/16) + j in a lane, which is the B operand of step j of
// O^T = V^T P^T (contraction index c = key 4c + j).  Operands come straight from memory (the caches hold
// them: 16 KB of K and V a tile at most).  One head, d = 64, 260 slots, chunks of 32: 114 us with one workgroup per
// row and scalar arithmetic, 11 with this.  Tiles at an edge look for values that are not finite, in a loop of their
// own: the same call 29.4 -> 30.1 us, 128 rows of 32 heads against 1K slots 129.3 either way; the test in the one loop cost the
// large launches 6 %.
constexpr int kF32Waves = 8;

template <int D>
__global__ __launch_bounds__(kF32Waves * 64) void attn_f32_kernel(Geom g, SegList sl, int Q, const float* __restrict__ Qr,
                                                                  const float* __restrict__ Kr, const float* __restrict__ Vc,
                                                                  const float* __restrict__ Krc, const float* __restrict__ Vch,
                                                                  float* __restrict__ out, float* __restrict__ lse2)
{
    constexpr int DB = D / 16, STR = D + 4;
    __shared__ __attribute__((aligned(16))) float osum[kF32Waves][16][STR];
    __shared__ float ms[kF32Waves][16], ls[kF32Waves][16];
    const int bh = blockIdx.y, b = bh / g.Hkv, hk = bh % g.Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, n = l & 15, c = l >> 4;
    const int r0 = blockIdx.x * 16, GQ = g.G * Q;
    const int r = min(r0 + n, GQ - 1), h = hk * g.G + r / Q, i = r % Q;      // this lane's query
    const int r_last = min(r0 + 15, GQ - 1);
    const bool one_head = r0 / Q == r_last / Q;
    const int imax = one_head ? r_last % Q : Q - 1, imin = one_head ? r0 % Q : 0;   // chunk keys after imax are seen by no row here, those up to imin by all
    const float sc = g.scale * kF32Log2e;

    f32x4_t o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;
    float q[D / 4];
    int first = 0, q_var = -1;                                               // first tile of the segment
    for (int si = 0; si < sl.n; ++si) {
        const Seg sg = sl.s[si];
        const int len = sg.chunk ? min(sg.len, imax + 1) : sg.len, nt = (len + kF32Keys - 1) / kF32Keys;
        const size_t row0 = sg.chunk ? (size_t)bh * Q : (size_t)bh * g.slots + sg.start;
        const float *kbase = (sg.chunk ? Krc : Kr) + row0 * D, *vbase = (sg.chunk ? Vch : Vc) + row0 * D;
        auto tile = [&](int t, auto edge) {                                  // edge: the end of the segment, or keys of the chunk that some row does not see
            if (sg.qvar != q_var) {
                q_var = sg.qvar;
                load_quarter<D>(Qr + ((((size_t)q_var * g.B + b) * g.Hq + h) * Q + i) * D, c, q);
            }
            const int k0 = t * kF32Keys;
            float k[D / 4], v[4][DB];
            load_quarter<D>(kbase + (size_t)min(k0 + n, len - 1) * D, c, k);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float* vr = vbase + (size_t)min(k0 + 4 * c + j, len - 1) * D + n;
#pragma unroll
                for (int db = 0; db < DB; ++db) v[j][db] = vr[16 * db];
            }
            f32x4_t s = product<D>(k, q) * sc;
            const int lim = (sg.chunk ? min(i, len - 1) : len - 1) - k0 - 4 * c;      // keys j <= lim are visible
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j > lim) s[j] = -INFINITY;
            const float mx = max_of_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
            if (__any(mx > m)) {
                const float mn = fmaxf(m, mx), alpha = m == mn ? 1.f : exp2f(m - mn);
                m = mn;
                lsum *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] *= alpha;
            }
            const float mr = m == -INFINITY ? 0.f : m;                       // a row that has seen no key yet
            if (decltype(edge)::value) {
                // a key that a row does not see has probability zero, but zero times an infinite or undefined value (a
                // later token's, or the last row's standing in for rows that do not exist) is not zero
                float not_finite = 0.f;
#pragma unroll
                for (int db = 0; db < DB; ++db) not_finite += v[3][db] * 0.f;                // (lanes that hold the last row's)
                if (sg.chunk) {
#pragma unroll
                    for (int db = 0; db < DB; ++db) not_finite += (v[0][db] * 0.f + v[1][db] * 0.f) + v[2][db] * 0.f;
                }
                if (__any(not_finite != 0.f)) {
                    float p[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        p[j] = exp2f(s[j] - mr);
                        lsum += p[j];
                    }
                    add_visible<D>(vbase, k0, sg.chunk ? min(len, i + 1) : len, n, c, p, o);
                    return;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float p = exp2f(s[j] - mr);
                lsum += p;
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j][db], p, o[db], 0, 0, 0);
            }
        };
        const int whole = (sg.chunk ? imin + 1 : len) / kF32Keys;            // tiles every row here sees whole
        int t = (wave + kF32Waves - first % kF32Waves) % kF32Waves;
        for (; t < whole; t += kF32Waves) tile(t, std::false_type());
        for (; t < nt; t += kF32Waves) tile(t, std::true_type());
        first += nt;
    }
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (c == 0) { ms[wave][n] = m; ls[wave][n] = lsum; }
#pragma unroll
    for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4_t*>(&osum[wave][n][16 * db + 4 * c]) = o[db];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 16 * D; idx += kF32Waves * 64) {
        const int row = idx / D, e = idx % D;
        if (r0 + row >= GQ) break;
        float mm = -INFINITY;
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) mm = fmaxf(mm, ms[w][row]);
        float a = 0.f, t = 0.f;
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            const float f = ms[w][row] == -INFINITY ? 0.f : exp2f(ms[w][row] - mm);
            a += f * osum[w][row][e];
            t += f * ls[w][row];
        }
        const int hh = (r0 + row) / Q, qi = (r0 + row) % Q;
        const size_t head = (size_t)b * g.Hq + hk * g.G + hh;
        out[(((size_t)b * Q + qi) * g.Hq + hk * g.G + hh) * D + e] = a / t;
        if (e == 0) lse2[head * Q + qi] = mm + log2f(t);
    }
}

// ------------------------------------------------------------------ score sums
//
// A workgroup owns 16 keys and keeps them as the B operand; its four waves share the 16-row blocks of the
// last `tail` query rows, head by head.  A lane holds one key and four rows of a block: the weighted
// probabilities (final normaliser from the attention kernel, base 2) are summed in the lane, over the lane groups, and
// over the waves in a fixed order.  (Same geometry as above: 194 us with one thread per key, 4.7 with this.)
constexpr int kF32ScoreWaves = 4;

template <int D>
__global__ __launch_bounds__(kF32ScoreWaves * 64) void score_f32_kernel(Geom g, SegList sl, int Q, int qstride, int tail, float decay,
                                                                        const float* __restrict__ Qr, const float* __restrict__ Kr,
                                                                        const float* __restrict__ Krc, const float* __restrict__ lse2,
                                                                        const float* __restrict__ wrow, float* __restrict__ mu,
                                                                        float* __restrict__ mu_chunk)
{
    __shared__ float part[2][kF32ScoreWaves][16];
    const int bh = blockIdx.y, b = bh / g.Hkv, hk = bh % g.Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, n = l & 15, c = l >> 4;
    int t = blockIdx.x, si = 0;
    for (; si < sl.n; ++si) {
        const int nt = (sl.s[si].len + kF32Keys - 1) / kF32Keys;
        if (t < nt) break;
        t -= nt;
    }
    if (si >= sl.n) return;
    const Seg sg = sl.s[si];
    const int key = t * kF32Keys + n;
    const size_t row0 = sg.chunk ? (size_t)bh * Q : (size_t)bh * g.slots + sg.start;
    float k[D / 4];
    load_quarter<D>((sg.chunk ? Krc : Kr) + (row0 + min(key, sg.len - 1)) * D, c, k);
    const float sc = g.scale * kF32Log2e;
    const int i_first = max(Q - tail, sg.chunk ? t * kF32Keys : 0);          // chunk keys are seen by their own and later rows
    float red = 0.f;
    for (int hh = 0; hh < g.G; ++hh) {
        const size_t head = (size_t)b * g.Hq + hk * g.G + hh;
        const float* qb = Qr + (((size_t)sg.qvar * g.B + b) * g.Hq + hk * g.G + hh) * (size_t)Q * D;
        float sum = 0.f;
        for (int i0 = i_first + wave * 16; i0 < Q; i0 += kF32ScoreWaves * 16) {
            float q[D / 4];
            load_quarter<D>(qb + (size_t)min(i0 + n, Q - 1) * D, c, q);
            float w[4], ls[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = min(i0 + 4 * c + j, Q - 1);
                w[j] = wrow[Q - 1 - i];
                ls[j] = lse2[head * Q + i];
            }
            const f32x4_t s = product<D>(q, k);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + 4 * c + j;
                if (i < Q && (!sg.chunk || key <= i)) sum += w[j] * exp2f(s[j] * sc - ls[j]);
            }
        }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        if (c == 0) part[hh & 1][wave][n] = sum;
        __syncthreads();                                                     // (two buffers: one barrier per head)
        if (wave == 0) {
            float total = 0.f;
#pragma unroll
            for (int x = 0; x < kF32ScoreWaves; ++x) total += part[hh & 1][x][n];
            if (g.head_reduce == CASCADE_REDUCE_MAX) red = hh == 0 ? total : fmaxf(red, total);
            else red += total;
        }
    }
    if (wave > 0 || c > 0 || key >= sg.len) return;
    if (g.head_reduce == CASCADE_REDUCE_MEAN) red /= (float)g.G;
    if (sg.chunk) mu_chunk[(size_t)bh * qstride + key] = red;
    else {
        float* p = mu + row0 + key;
        *p = decay * *p + red;
    }
}

// fp32 with a head dimension the MFMA kernels are written for; everything else takes the scalar kernels
bool attn_f32_ok(const Geom& g, int dtype) { return dtype == CASCADE_F32 && (g.d == 64 || g.d == 128); }

void launch_attn_f32(const Geom& g, const DevBuffers& b, const SegList& sl, int Q, void* out, hipStream_t s)
{
    const dim3 grid((g.G * Q + 15) / 16, g.B * g.Hkv), block(kF32Waves * 64);
#define CKV_ATTN_F32(D)                                                                                                          \
    hipLaunchKernelGGL(attn_f32_kernel<D>, grid, block, 0, s, g, sl, Q, (const float*)b.Qr, (const float*)b.Kr, (const float*)b.Vc, \
                       (const float*)b.Krc, (const float*)b.Vch, (float*)out, b.lse)
    if (g.d == 128) CKV_ATTN_F32(128); else CKV_ATTN_F32(64);
#undef CKV_ATTN_F32
}

void launch_score_f32(const Geom& g, const DevBuffers& b, const SegList& sl, int Q, int max_chunk, int tail_rows, float decay, hipStream_t s)
{
    int tiles = 0;
    for (int i = 0; i < sl.n; ++i) tiles += (sl.s[i].len + kF32Keys - 1) / kF32Keys;
    const dim3 grid(tiles, g.B * g.Hkv), block(kF32ScoreWaves * 64);
#define CKV_SCORE_F32(D)                                                                                                          \
    hipLaunchKernelGGL(score_f32_kernel<D>, grid, block, 0, s, g, sl, Q, max_chunk, tail_rows, decay, (const float*)b.Qr,            \
                       (const float*)b.Kr, (const float*)b.Krc, b.lse, b.wrow, b.mu, b.mu_chunk)
    if (g.d == 128) CKV_SCORE_F32(128); else CKV_SCORE_F32(64);
#undef CKV_SCORE_F32
}

}  // namespace ckv
