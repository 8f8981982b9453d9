// Chunk attention and score sums in fp32 on the matrix cores (head dimension 64 or 128): the fp32
// configuration.  The arithmetic is fp32 throughout; v_mfma_f32_16x16x4_f32 takes fp32 operands.
//
// v_mfma_f32_16x16x4_f32, D[m][n] += sum_k A[m][k] B[k][n]: lane l holds A[l%16][l/16] and
// B[l/16][l%16]; D: column l%16, rows 4*(l/16) .. +3.  Which element of the head dimension a
// contraction index means is free as long as A and B agree: lane group c = l/16 takes elements
// c*D/4 + step, so a lane reads D/4 contiguous floats of its row.
#include <algorithm>

#include "launch.h"
#include "mfma_util.h"
#include "plan_core.h"

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
#pragma nounroll
    for (int x = 0; x < kF32Keys; ++x) {
        const int j = x & 3;
        const float px = __shfl(j == 0 ? p[0] : j == 1 ? p[1] : j == 2 ? p[2] : p[3], (x >> 2) * 16 + n, 64);   // key x of this lane's row
        if (k0 + x >= end) continue;
        const float* v = vbase + (size_t)(k0 + x) * D + 4 * c * (D / 16);
#pragma unroll
        for (int db = 0; db < D / 16; ++db)
#pragma unroll
            for (int y = 0; y < 4; ++y) o[db][y] += v[y * (D / 16) + db] * px;
    }
}

// ------------------------------------------------------------------ attention
//
// A workgroup owns 16 (head, token) rows of one KV head; its eight or sixteen waves take the 16-key tiles in turn,
// each with its own running maximum, and are combined at the end: small launches, which is what this
// configuration is for, are bound by the latency of one wave's tiles, so the keys are spread over waves.
// S^T = K Q^T leaves query l%16 and keys 4*(l/16) + j in a lane, which is the B operand of step j of
// O^T = V^T P^T (contraction index c = key 4c + j).  Row m of block db of O^T is element m D/16 + db, so that a lane reads its
// elements of a row of V in 16-byte pieces (one by one, the loads of a tile were twice as many instructions, and what bound it).  Operands come straight from memory (the caches hold
// them: 16 KB of K and V a tile at most).  One head, d = 64, 260 slots, chunks of 32: 114 us with one workgroup per
// row and scalar arithmetic, 11.4 with this, which is a chain of latencies (segments, operands, products, the waves'
// results; one fp32 MFMA takes a SIMD 32 cycles).  Tiles at an edge look for values that are not finite.
//
// Launches that leave compute units without work divide a row block's tiles over workgroups as well (SPLIT, f32_splits), each
// with a partial result that merge_f32_kernel combines.  Against one workgroup a row block, V element by element and the segments
// read one after the other, us a call: d = 64, one head, chunks of 32: 260 slots 30.1 -> 25.7 (with the update in one launch), 16K slots
// 271 -> 52; d = 128, one head, one row on 16K slots 554 -> 53; 128 rows of 32 heads on 1K slots 130 -> 123.  67 forms: 1.005 at least, 1.58 in the median.
// The bound on registers (128 at d = 64) lets a CU hold two workgroups of eight waves.  It spills four to six registers, outside the
// loop over the tiles; with 138 registers, none spilled and one workgroup a CU, 320 row blocks on 192 slots took 63.7 us a call
// instead of 60.1, 1024 on 128 slots 88.5 instead of 80.2.

// The segments cut into 16-key tiles: first tile of every segment (INT32_MAX behind the last, which is the chunk).
struct F32Tiles {
    int total;
    int first[kMaxSegments];
};

template <int D, bool SPLIT, int WAVES>
__global__ __launch_bounds__(WAVES * 64, D == 64 ? 4 : 2) void attn_f32_kernel(Geom g, SegList sl, F32Tiles ft, int Q, int n_split, const float* __restrict__ Qr,
                                                                  const float* __restrict__ Kr, const float* __restrict__ Vc,
                                                                  const float* __restrict__ Krc, const float* __restrict__ Vch,
                                                                  float* __restrict__ out, float* __restrict__ lse2, float* __restrict__ part)
{
    constexpr int DB = D / 16, STR = D + 4;
    __shared__ __attribute__((aligned(16))) float osum[WAVES][16][STR];
    __shared__ float ms[WAVES][16], ls[WAVES][16], fs[WAVES][16], top[16];
    const int bh = blockIdx.y, b = bh / g.Hkv, hk = bh % g.Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, n = l & 15, c = l >> 4;
    // the segments, one per lane: one load, and no other between two tiles
    const int li = min(l, kMaxSegments - 1), li_first = ft.first[li], seg_first = l < kMaxSegments ? li_first : INT32_MAX;
    const Seg my = sl.s[li];
    const int r0 = blockIdx.x * 16, GQ = g.G * Q;
    const int r = min(r0 + n, GQ - 1), h = hk * g.G + r / Q, i = r % Q;      // this lane's query
    const int r_last = min(r0 + 15, GQ - 1);
    const bool one_head = r0 / Q == r_last / Q;
    const int imax = one_head ? r_last % Q : Q - 1, imin = one_head ? r0 % Q : 0;   // chunk keys after imax are seen by no row here, those up to imin by all
    const float sc = g.scale * kF32Log2e;
    int t0 = 0, t1 = ft.first[sl.n - 1] + imax / kF32Keys + 1;               // tiles of this row block (the chunk is the last segment), of this split
    if (SPLIT) {
        const int all = t1;
        t0 = share_begin(all, (int)blockIdx.z, n_split);
        t1 = share_begin(all, (int)blockIdx.z + 1, n_split);
    }

    f32x4_t o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;
    float q[D / 4];
    int q_var = -1;
    for (int next = t0 + wave; next < t1;) {                                 // (the segments in which the wave has tiles)
        const int si = __builtin_popcountll(__ballot(next >= seg_first)) - 1, first = __builtin_amdgcn_readlane(seg_first, si);
        const Seg sg = {__builtin_amdgcn_readlane(my.start, si), __builtin_amdgcn_readlane(my.len, si), __builtin_amdgcn_readlane(my.qvar, si),
                        __builtin_amdgcn_readlane(my.chunk, si)};
        const int len = sg.chunk ? min(sg.len, imax + 1) : sg.len, nt = (len + kF32Keys - 1) / kF32Keys;
        const size_t row0 = sg.chunk ? (size_t)bh * Q : (size_t)bh * g.slots + sg.start;
        const float *kbase = (sg.chunk ? Krc : Kr) + row0 * D, *vbase = (sg.chunk ? Vch : Vc) + row0 * D;
        auto tile = [&](int t, bool edge) {                                  // edge: the end of the segment, or keys of the chunk that some row does not see
            if (sg.qvar != q_var) {
                q_var = sg.qvar;
                load_quarter<D>(Qr + ((((size_t)q_var * g.B + b) * g.Hq + h) * Q + i) * D, c, q);
            }
            const int k0 = t * kF32Keys;
            float k[D / 4], v[4][DB];
            load_quarter<D>(kbase + (size_t)min(k0 + n, len - 1) * D, c, k);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float* vr = vbase + (size_t)min(k0 + 4 * c + j, len - 1) * D + n * DB;
#pragma unroll
                for (int db = 0; db < DB; db += 4) *reinterpret_cast<f32x4_t*>(&v[j][db]) = *reinterpret_cast<const f32x4_t*>(vr + db);
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
            if (edge) {
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
        const int end = min(nt, t1 - first), whole = min((sg.chunk ? imin + 1 : len) / kF32Keys, end);   // tiles every row here sees whole
        int t = next - first;
#pragma nounroll                                   // (one copy of the code: a small launch is bound by fetching it)
        for (; t < end; t += WAVES) tile(t, t >= whole);
        next = first + t;
    }
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (c == 0) { ms[wave][n] = m; ls[wave][n] = lsum; }
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
        for (int db = 0; db < DB; db += 4)
            *reinterpret_cast<f32x4_t*>(&osum[wave][n][(4 * c + y) * DB + db]) = f32x4_t{o[db][y], o[db + 1][y], o[db + 2][y], o[db + 3][y]};
    __syncthreads();
    // what the waves' results of a row are multiplied by, once for all its elements
    const int fw = threadIdx.x / 16, fr = threadIdx.x % 16;
    float mm = -INFINITY;
    if (fw < WAVES) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mm = fmaxf(mm, ms[w][fr]);
        fs[fw][fr] = ms[fw][fr] == -INFINITY ? 0.f : exp2f(ms[fw][fr] - mm);
        if (fw == 0) top[fr] = mm;
    }
    __syncthreads();
#pragma nounroll
    for (int idx = threadIdx.x; idx < 16 * D; idx += WAVES * 64) {
        const int row = idx / D, e = idx % D;
        if (r0 + row >= GQ) break;
        float a = 0.f, t = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            a += fs[w][row] * osum[w][row][e];
            t += fs[w][row] * ls[w][row];
        }
        if (SPLIT) {
            const size_t prow = ((size_t)blockIdx.z * gridDim.y + bh) * GQ + r0 + row;
            part[prow * (D + 2) + e] = a;
            if (e == 0) { part[prow * (D + 2) + D] = top[row]; part[prow * (D + 2) + D + 1] = t; }
            continue;
        }
        const int hh = (r0 + row) / Q, qi = (r0 + row) % Q;
        const size_t head = (size_t)b * g.Hq + hk * g.G + hh;
        out[(((size_t)b * Q + qi) * g.Hq + hk * g.G + hh) * D + e] = a / t;
        if (e == 0) lse2[head * Q + qi] = top[row] + log2f(t);
    }
}

// The splits' results of a row combined: D threads a row, the splits in order.
template <int D>
__global__ __launch_bounds__(256) void merge_f32_kernel(Geom g, int Q, int n_split, const float* __restrict__ part, float* __restrict__ out,
                                                        float* __restrict__ lse2)
{
    const int bh = blockIdx.y, b = bh / g.Hkv, hk = bh % g.Hkv, r = blockIdx.x * (256 / D) + threadIdx.x / D, e = threadIdx.x % D;
    const int rows = g.G * Q;
    if (r >= rows) return;
    const size_t stride = (size_t)gridDim.y * rows * (D + 2);
    const float* p = part + ((size_t)bh * rows + r) * (D + 2);
    float mm = -INFINITY;
    for (int s = 0; s < n_split; ++s) mm = fmaxf(mm, p[s * stride + D]);
    float a = 0.f, t = 0.f;
    for (int s = 0; s < n_split; ++s) {
        const float m = p[s * stride + D], f = m == -INFINITY ? 0.f : exp2f(m - mm);   // (a split without a key of this row)
        a += f * p[s * stride + e];
        t += f * p[s * stride + D + 1];
    }
    const int hh = r / Q, qi = r % Q;
    out[(((size_t)b * Q + qi) * g.Hq + hk * g.G + hh) * D + e] = a / t;
    if (e == 0) lse2[((size_t)b * g.Hq + hk * g.G + hh) * Q + qi] = mm + log2f(t);
}

// ------------------------------------------------------------------ score sums
//
// A workgroup owns 16 keys and keeps them as the B operand; its four waves share the 16-row blocks of the
// last `tail` query rows, head by head.  A lane holds one key and four rows of a block: the weighted
// probabilities (final normaliser from the attention kernel, base 2) are summed in the lane, over the lane groups, and
// over the waves in a fixed order.  (Same geometry as above: 194 us with one thread per key, 4.7 with this.)
constexpr int kF32ScoreWaves = 4;

template <int D>
__global__ __launch_bounds__(kF32ScoreWaves * 64) void score_f32_kernel(Geom g, SegList sl, F32Tiles ft, int Q, int qstride, int tail, float decay,
                                                                        const float* __restrict__ Qr, const float* __restrict__ Kr,
                                                                        const float* __restrict__ Krc, const float* __restrict__ lse2,
                                                                        const float* __restrict__ wrow, float* __restrict__ mu,
                                                                        float* __restrict__ mu_chunk)
{
    __shared__ float part[2][kF32ScoreWaves][16];
    const int bh = blockIdx.y, b = bh / g.Hkv, hk = bh % g.Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, n = l & 15, c = l >> 4;
    const int si = table_entry(ft.first, (int)blockIdx.x), t = (int)blockIdx.x - ft.first[si];
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

static F32Tiles f32_tiles(const SegList& sl)
{
    F32Tiles ft;
    ft.total = 0;
    for (int i = 0; i < kMaxSegments; ++i) {
        ft.first[i] = i < sl.n ? ft.total : INT32_MAX;
        if (i < sl.n) ft.total += (sl.s[i].len + kF32Keys - 1) / kF32Keys;
    }
    return ft;
}

// Workgroups that share the tiles of a row block: while there are fewer than 256 workgroups and each keeps
// kF32SplitTiles tiles, as far as the partial results fit memory that is free at that time (DevBuffers::f32_part).
constexpr int kF32SplitTiles = 32;
static int f32_splits(const Geom& g, const DevBuffers& b, int rows, int tiles)
{
    const int wgs = (rows + 15) / 16 * g.B * g.Hkv;
    const size_t room = b.f32_part_floats / ((size_t)g.B * g.Hkv * rows * (g.d + 2));
    const int n = (int)std::min<size_t>(std::min(256 / wgs, tiles / kF32SplitTiles), room);
    return n < 1 ? 1 : n;
}

void launch_attn_f32(const Geom& g, const DevBuffers& b, const SegList& sl, int Q, void* out, hipStream_t s)
{
    const F32Tiles ft = f32_tiles(sl);
    const int rows = g.G * Q, n_split = f32_splits(g, b, rows, ft.total);
    const dim3 grid((rows + 15) / 16, g.B * g.Hkv, n_split);
    float* part = b.f32_part;
#define CKV_ATTN_F32(D, SPLIT, WAVES)                                                                                                           \
    hipLaunchKernelGGL((attn_f32_kernel<D, SPLIT, WAVES>), grid, dim3(WAVES * 64), 0, s, g, sl, ft, Q, n_split, (const float*)b.Qr,               \
                       (const float*)b.Kr, (const float*)b.Vc, (const float*)b.Krc, (const float*)b.Vch, (float*)out, b.lse, part)
#define CKV_MERGE_F32(D)                                                                                                                        \
    hipLaunchKernelGGL(merge_f32_kernel<D>, dim3((rows + 256 / D - 1) / (256 / D), g.B * g.Hkv), dim3(256), 0, s, g, Q, n_split, part, (float*)out, b.lse)
    // sixteen waves where that many fit a compute unit's registers (d = 64) and the launch leaves compute units without work
    const bool many = (long)grid.x * grid.y * n_split <= 256;
    if (g.d == 128) { if (n_split > 1) CKV_ATTN_F32(128, true, 8); else CKV_ATTN_F32(128, false, 8); }
    else if (many) { if (n_split > 1) CKV_ATTN_F32(64, true, 16); else CKV_ATTN_F32(64, false, 16); }
    else CKV_ATTN_F32(64, false, 8);         // (not split: there are more than 256 row blocks)
    if (n_split > 1) { if (g.d == 128) CKV_MERGE_F32(128); else CKV_MERGE_F32(64); }
#undef CKV_MERGE_F32
#undef CKV_ATTN_F32
}

void launch_score_f32(const Geom& g, const DevBuffers& b, const SegList& sl, int Q, int max_chunk, int tail_rows, float decay, hipStream_t s)
{
    const F32Tiles ft = f32_tiles(sl);
    const dim3 grid(ft.total, g.B * g.Hkv), block(kF32ScoreWaves * 64);
#define CKV_SCORE_F32(D)                                                                                                          \
    hipLaunchKernelGGL(score_f32_kernel<D>, grid, block, 0, s, g, sl, ft, Q, max_chunk, tail_rows, decay, (const float*)b.Qr,            \
                       (const float*)b.Kr, (const float*)b.Krc, b.lse, b.wrow, b.mu, b.mu_chunk)
    if (g.d == 128) CKV_SCORE_F32(128); else CKV_SCORE_F32(64);
#undef CKV_SCORE_F32
}

}  // namespace ckv
