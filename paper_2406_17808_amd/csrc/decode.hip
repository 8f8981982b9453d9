// Decode step (Eq. 2): one query per sequence against the whole cache plus its own key.
//
// Two launches.  decode_attend streams K and V once: every split of the cached rows leaves its
// logits, its maximum, its sum of exponentials and its unnormalised output.  decode_finish
// combines the splits, takes the EMA step of every cached row's score (Section 3.1; it needs the
// final normaliser, hence the logits, 16 bytes per cached row at 4 query heads per KV head, that
// pass through a scratch array) and inserts the token.  Logits are base-2 exponents: the queries
// carry the softmax scale and log2(e).
#include "async_copy.h"
#include "launch.h"
#include "row_ops.h"

namespace ckv {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kDecRows = kDecodeTileRows;
constexpr int kMaxG = 8;
constexpr float kLog2e = 1.4426950408889634f;

// Logits of a step: [B*Hkv][tile][32 * MAXG] floats, MAXG = group size rounded up
// to 1, 2, 4 or 8 (decode_logit_heads).  Row 16 gi + 4 c + j of a tile and head n sit at
// ((gi * MAXG + n) * 4 + c) * 4 + j, the order in which the accumulators of the QK product hold them:
// four rows of one head are 16 adjacent bytes for the kernel that writes them and the one that reads them.
template <int MAXG> __device__ inline int logit_index(int row, int n)
{
    return (((row >> 4) * MAXG + n) * 4 + ((row >> 2) & 3)) * 4 + (row & 3);
}

// A reduction over the wave in registers (all lanes get the result): two lane swaps, then rotations inside the rows of 16
// lanes; a shuffle through the LDS crossbar takes about as long as all six steps.
template <typename Op> __device__ inline float wave_reduce(float x, Op op)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(b[0]), __uint_as_float(b[1]));
    constexpr int kRowRor = 0x120;
    x = op(x, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), kRowRor + 8, 0xf, 0xf, false)));
    x = op(x, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), kRowRor + 4, 0xf, 0xf, false)));
    x = op(x, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), kRowRor + 2, 0xf, 0xf, false)));
    return op(x, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), kRowRor + 1, 0xf, 0xf, false)));
}
__device__ inline float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ inline float wave_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }

// The runs of a step, one per lane: one load for all of them and a vote find the run of a tile, where a walk over the
// list costs a scalar load per run, one after the other (at the start of a workgroup, with cold caches).
struct LaneRuns {
    int tile0, start, len, rot;
    __device__ LaneRuns(const DecodeRuns& r)
    {
        const int l = threadIdx.x & 63, i = min(l, kMaxDecodeRuns - 1);
        const int first = r.tile0[i];
        tile0 = l < kMaxDecodeRuns ? first : INT32_MAX;
        start = r.start[i];
        len = r.len[i];
        rot = r.rot[i];
    }
};

// The splits of a step: the first `more` have each + 1 tiles, the others each.  (Divided on the host: 64-bit divisions at the
// start of a workgroup are 300 instructions fetched with a cold cache.)
struct Splits {
    int n, each, more;
};

// A wave's position among the tiles.  All fields are the same in all lanes.
struct TileWalk {
    int tile, next0;                   // tile; the first tile behind its run
    int tile0, start0, len, rot;       // of its run
    int start, nvalid;                 // first slot and rows of the tile
    __device__ void seek(const LaneRuns& u, int to)
    {
        tile = to;
        const int i = __builtin_popcountll(__ballot(tile >= u.tile0)) - 1;
        tile0 = __builtin_amdgcn_readlane(u.tile0, i);
        start0 = __builtin_amdgcn_readlane(u.start, i);
        len = __builtin_amdgcn_readlane(u.len, i);
        rot = __builtin_amdgcn_readlane(u.rot, i);
        next0 = tile0 + (len + kDecRows - 1) / kDecRows;
        place();
    }
    __device__ void place()
    {
        const int r0 = (tile - tile0) * kDecRows;
        start = start0 + r0;
        nvalid = min(kDecRows, len - r0);
    }
    template <typename Runs> __device__ void advance(const Runs& u, int by)    // (DecodeRuns: loaded anew where a run ends)
    {
        if (tile + by >= next0) seek(u, tile + by);      // (past the last tile: its run, and nothing that is read)
        else { tile += by; place(); }
    }
};

// (max, sum of exp2) pairs combine associatively
__device__ inline void ml_merge(float& m, float& l, float m2, float l2)
{
    if (l2 > 0.f) {
        const float mn = fmaxf(m, m2);
        l = l * __builtin_amdgcn_exp2f(m - mn) + l2 * __builtin_amdgcn_exp2f(m2 - mn);
        m = mn;
    }
}

// What sums relative to maximum m are multiplied by when the maximum becomes mn; the maximum exponents are taken
// against.  (Logits that overflowed to -infinity are keys of probability zero, also where nothing else was seen yet.)
__device__ inline float rescale_of(float m, float mn) { return m == mn ? 1.f : __builtin_amdgcn_exp2f(m - mn); }
__device__ inline float finite_max(float m) { return m == -INFINITY ? 0.f : m; }

// The step's partial results: part[(b, query head)][split] = (maximum, sum), one more entry for the token's own
// key (its logit, 1); opart[(b, query head)][split][d] unnormalised.
__device__ inline float* part_of(float* part, size_t head, int n_splits, int split) { return part + (head * (n_splits + 1) + split) * 2; }

// The own key: <R(n) q, R(n) k> = <q, k>.  One wave per head of the group (heads wave, wave + WAVES, ..); load() early,
// finish() when there is nothing better to do.  WAVES of the workgroup take part.  (Whole words, as they are in memory, in between: what is converted after a
// load is waited for there.)
__device__ inline float word_product(const float*, uint32_t a, uint32_t b) { return __uint_as_float(a) * __uint_as_float(b); }
__device__ inline float word_product(const bf16_t*, uint32_t a, uint32_t b)
{
    return __uint_as_float(a << 16) * __uint_as_float(b << 16) + __uint_as_float(a & 0xFFFF0000u) * __uint_as_float(b & 0xFFFF0000u);
}
template <typename T, int D, int WAVES>
struct OwnLogits {
    static constexpr int NH = kMaxG / WAVES, kWords = D * (int)sizeof(T) / 4, NE = (kWords + 63) / 64;
    uint32_t qe[NH][NE], ke[NE];
    __device__ void load(const Geom& g, int b, int hk, const T* __restrict__ q, const T* __restrict__ k_new)
    {
        const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
        const uint32_t* kw = reinterpret_cast<const uint32_t*>(k_new + ((size_t)b * g.Hkv + hk) * D);
#pragma unroll
        for (int x = 0; x < NE; ++x) {
            const int w = min(x * 64 + l, kWords - 1);
            ke[x] = kw[w];
#pragma unroll
            for (int i = 0; i < NH; ++i) {
                const int hh = min(wave + i * WAVES, g.G - 1);
                qe[i][x] = reinterpret_cast<const uint32_t*>(q + ((size_t)b * g.Hq + hk * g.G + hh) * D)[w];
            }
        }
    }
    __device__ void finish(const Geom& g, int b, int hk, float qscale, float* __restrict__ part, int n_splits) const
    {
        const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const int hh = wave + i * WAVES;
            if (hh >= g.G) break;
            float acc = 0.f;
#pragma unroll
            for (int x = 0; x < NE; ++x) acc += x * 64 + l < kWords ? word_product((const T*)nullptr, qe[i][x], ke[x]) : 0.f;
            acc = wave_sum(acc);
            if (l == 0) {
                float* p = part_of(part, (size_t)b * g.Hq + hk * g.G + hh, n_splits, n_splits);
                p[0] = acc * qscale;
                p[1] = 1.f;
            }
        }
    }
};

// ------------------------------------------------------------------ attend, bf16: MFMA fed from LDS
//
// v_mfma_f32_16x16x32_bf16: for lane l, A holds row l%16, B column l%16, both with the 8
// contraction indices 8*(l/16)..+7; D holds column l%16, rows 4*(l/16)..+3.  S = K Q^T: rows are 16
// keys, columns the query heads of the group (padded with zeros to 16).  A lane then holds, for head
// n = l%16, the keys 4c + {0..3} and 16 + 4c + {0..3} of the tile (c = l/16), and that is taken as the
// contraction order of O^T = V^T P^T: the exponentials of the accumulators ARE the B operand, no
// probability crosses a lane, and the A operand (8 rows of one column of V) is two transposing reads
// (ds_read_b64_tr_b16) of rows 4c .. 4c+3 and 16 + 4c .. +3.
//
// Every wave streams its own tiles through a private ring of LDS stages (K and V of DEPTH tiles) filled by asynchronous
// copies, 128 KB a workgroup, so that most of it is in flight whatever the waves compute, and no workgroup barrier is needed
// inside the loop.  A wave keeps its own running maximum per head, raised only when a tile exceeds it by 2^8 (most tiles
// then leave the accumulators alone).  Eight waves: a step on a cache of 256 tiles a KV head or less is then one tile a
// wave, all of them computed at the same time; with four waves of two tiles the second waited for the first, and the compiler
// (one wave a SIMD, 512 registers) kept the accumulators in the other half of the register file and copied them
// back and forth for every tile.
//
// Bound by memory where the cache is large, by the latency of one tile where it is small.  At 8K slots and 8 KV heads a
// workgroup ended 10.0 us after it began: 3.4 until its last copy was issued (a scalar load for every run in the list, two
// 64-bit divisions), 1.5 for queries that came behind the tiles, 2.2 for the second tile, 2.0 where a wave had a third;
// now 6.0, in the splits with a tile more 7.1.  us a step with decode_finish, timed as calls of a program, before and after: 8K
// slots 19.1 -> 14.2, a layer of 4K slots 16.2 -> 11.9 (where the host's calls are the limit), 8 sequences of 16K slots 109.6 ->
// 103.8 (with the logits written tile by tile).
//
// On a large cache the logits cost far more than their bytes: without their stores (a sixteenth of the bytes read,
// for groups of 4) a step of 32 sequences of 65K slots took 1312 us, with them 1660: memory turns round for every
// few of them.  So a wave keeps the logits of HOLD tiles in registers and writes them at once, past the L2, which would put
// the lines out one by one later on: 8 tiles 1607, 16 tiles 1565, 32 tiles (R = 8) 1520, 40 to 48 the same; 32 tiles by way
// of the L2 1623 (groups of 4; R = 8 holds 128, 64 and 16 tiles for groups of 1, 2 and 8).  8 sequences of 16K slots 105.4 -> 95.5.
// (These are steps in a stream of steps; calls of a program with 8K slots take 1 us more.)  No lane is moved for it: the queries stand in all column groups of
// the product, so each group of MAXG columns keeps the tile that is its turn.  Where no wave has more tiles than one
// register holds, R = 1 does it, which is 0.4 to 0.8 us less (8K slots 13.9 -> 13.2, before 13.1; 32 sequences, 40
// tiles a workgroup, one head a KV head 35.4 -> 34.3); its few stores go through the L2 but for groups of 8 (one head 34.2 us
// against 34.7 past it, 8 heads 47.6 against 46.8).
//
// The piece permutations (16-byte pieces of a staged row): the 16 rows of a K fragment read, and the
// 8 rows one half of a wave reads in a transposing read, fall into different banks.
template <int D> struct DecSwizzle;
template <> struct DecSwizzle<128> {
    __device__ static int k(int row) { return row & 15; }
    __device__ static int v(int row) { return 2 * (row & 7); }
};
template <> struct DecSwizzle<64> {
    __device__ static int k(int row) { return (row >> 1) & 7; }
    __device__ static int v(int row) { return 2 * ((row >> 1) & 3); }
};

typedef __attribute__((ext_vector_type(8))) __bf16 dbf16x8_t;
typedef __attribute__((ext_vector_type(4))) float df32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t du32x4_t;
union DFrag {
    dbf16x8_t v;
    du32x4_t u;
};

__device__ inline uint32_t dec_pack_bf16(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) __bf16 b2;
    typedef __attribute__((ext_vector_type(2))) float f2;
    const f2 x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, b2));
}

typedef short dec_v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) dec_v4i16_t dec_lds_v4i16_t;

// ds_read_b64_tr_b16: the 16 lanes of a group address a 4-row x 16-column block of 16-bit
// elements (lane i: row i/4, columns 4*(i%4)..+3); lane i receives column i of the 4 rows.
__device__ inline uint2 read_tr16(const unsigned char* p)
{
    const dec_v4i16_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dec_lds_v4i16_t*)p);
    return __builtin_bit_cast(uint2, r);
}

// maximum over the four lanes that hold one head's keys (l, l^16, l^32, l^48)
__device__ inline float max_groups(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// the same sum
__device__ inline float sum_groups(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

constexpr float kDecRescale = 8.f;

constexpr int kAttendThreads = 512;
constexpr int kAttendWaves = kAttendThreads / 64;

template <int D, int MAXG, int R>
__global__ __launch_bounds__(kAttendThreads, 1) void decode_attend_kernel(
    Geom g, DecodeRuns runs, Splits sp, float qscale, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k_new,
    const bf16_t* __restrict__ Kr, const bf16_t* __restrict__ Vc, const float2* __restrict__ rope, float* __restrict__ logits,
    float* __restrict__ part, float* __restrict__ opart)
{
    constexpr int KS = D / 32;                     // MFMA steps over the head dimension (QK)
    constexpr int DB = D / 16;                     // MFMA row blocks over the head dimension (PV)
    constexpr int PPR = D / 8;                     // 16-byte pieces per row
    constexpr int RPI = 64 / PPR;                  // rows per copy instruction
    constexpr int kStage = kDecRows * D * 2;       // bytes of a staged K or V tile
    constexpr int NC = kStage / 1024;              // copies per stage
    constexpr int P = 16 / MAXG, HOLD = P * R;         // tiles whose logits share a register, tiles a wave holds
    constexpr int NS = 2 * R;                      // stores when all of them leave
    constexpr bool kThrough = R > 1 || MAXG == 8;  // whether they pass the L2 by
    constexpr int NQ = (MAXG * D * 2 + 1023) / 1024;   // copies that bring the group's queries
    constexpr int W = kAttendWaves, DEPTH = 8192 / kStage;
    constexpr int kLds = 160 * 1024, kFixed = W * DEPTH * 2 * kStage + W * (NQ * 1024 + D * 4) + W * 16 * 8;
    // Where there is room, a stage more for one tile: that of the first wave in splits of W * DEPTH + 1 tiles, which is what a
    // cache of a power of two of rows, sinks and ragged runs leaves in some of them.  Waiting for a stage to become
    // free cost those workgroups 2.5 of 9 us.
    constexpr bool kSpare = kFixed + 2 * kStage <= kLds;
    static_assert(kFixed <= kLds, "LDS");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[W][DEPTH][2][kStage];   // K and V of a tile
    __shared__ __attribute__((aligned(1024))) unsigned char spare[kSpare ? 2 : 1][kSpare ? kStage : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char qbuf[W][NQ * 1024];          // every wave's own copy of the group's queries
    __shared__ __attribute__((aligned(1024))) unsigned char csbuf[W][D * 4];             // (cos, sin) for its first tile
    __shared__ __attribute__((aligned(16))) float2 red[16][W];                           // (maximum, sum) of every head and wave
    static_assert(sizeof(float) * MAXG * D <= sizeof(ring[0]), "the partial outputs reuse the ring");
    const LaneRuns lr(runs);
    const int n_tiles = runs.n_tiles, n_splits = sp.n;
    const int split = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
    const int bh = b * g.Hkv + hk;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, n = l & 15, c = l >> 4;
    // this split's tiles; the waves take them in turn
    const int t_first = split * sp.each + min(split, sp.more), t_end = t_first + sp.each + (split < sp.more ? 1 : 0);
    const bf16_t* kbh = Kr + (size_t)bh * g.slots * D;
    const bf16_t* vbh = Vc + (size_t)bh * g.slots * D;
    const uint32_t ring_lds = lds_address(&ring[wave][0][0][0]), spare_lds = lds_address(&spare[0][0]);
    const unsigned char* ring_w = &ring[wave][0][0][0];
    const bool has_spare = kSpare && wave == 0 && t_end - t_first == W * DEPTH + 1;    // its last tile lies there

    int k_off[NC], v_off[NC], c_row[NC];           // what this lane copies of a stage: row and byte offset inside it
#pragma unroll
    for (int x = 0; x < NC; ++x) {
        c_row[x] = x * RPI + l / PPR;
        k_off[x] = ((l % PPR) ^ DecSwizzle<D>::k(c_row[x])) * 16;
        v_off[x] = ((l % PPR) ^ DecSwizzle<D>::v(c_row[x])) * 16;
    }
    auto issue = [&](const bf16_t* base, const int (&off)[NC], const TileWalk& t, uint32_t to) {
        const bf16_t* src = base + (size_t)t.start * D;
#pragma unroll
        for (int x = 0; x < NC; ++x)               // rows past the end repeat the last one
            async_copy_1k_stream(src, (uint32_t)(min(c_row[x], t.nvalid - 1) * (D * 2) + off[x]),
                                 __builtin_amdgcn_readfirstlane(to + (uint32_t)(x * 1024)));
    };

    TileWalk prod, cons;
    prod.seek(lr, t_first + wave);
    cons = prod;
    OwnLogits<bf16_t, D, W> own;
    if (split == 0) own.load(g, b, hk, q, k_new);
    // The queries and the row of (cos, sin) that turns them for the first tile come ahead of the tiles, by
    // the same kind of copies: ordinary loads would be waited for behind all the tiles.
    if (prod.tile < t_end) {
        const bf16_t* qg = q + ((size_t)b * g.Hq + hk * g.G) * D;
        const uint32_t q_lds = lds_address(&qbuf[wave][0]), q_last = (uint32_t)(g.G * D * 2 - 16);
        if (((uintptr_t)q & 15) == 0) {
#pragma unroll
            for (int x = 0; x < NQ; ++x)
                async_copy_1k(qg, min((uint32_t)(x * 1024 + l * 16), q_last), __builtin_amdgcn_readfirstlane(q_lds + x * 1024));
        } else {                                   // (a caller's tensor need not start where such a copy can)
#pragma unroll
            for (int x = 0; x < NQ; ++x)
                *reinterpret_cast<du32x4_t*>(&qbuf[wave][x * 1024 + l * 16]) =
                    *reinterpret_cast<const du32x4_t*>(reinterpret_cast<const unsigned char*>(qg) + min((uint32_t)(x * 1024 + l * 16), q_last));
        }
        if (l * 16 < D * 4)                        // (half of the wave, or a quarter)
            async_copy_1k(rope + (size_t)prod.rot * (D / 2), (uint32_t)(l * 16), __builtin_amdgcn_readfirstlane(lds_address(&csbuf[wave][0])));
    }
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (prod.tile < t_end) {
            issue(kbh, k_off, prod, ring_lds + (2 * i) * kStage);
            issue(vbh, v_off, prod, ring_lds + (2 * i + 1) * kStage);
            prod.advance(lr, W);
        }
    if (has_spare) {
        issue(kbh, k_off, prod, spare_lds);
        issue(vbh, v_off, prod, spare_lds + kStage);
        prod.advance(lr, W);
    }

    // fragment reads of this lane.  K: row 16 gi + n, piece 4 ks + c.  V: row 16 hf + 4 c + n / 4, 8 bytes
    // at element 16 db + 4 (n % 4)
    int a_off[2][KS], t_off[2], t_sw[2];
#pragma unroll
    for (int gi = 0; gi < 2; ++gi) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a_off[gi][ks] = (16 * gi + n) * (D * 2) + (((4 * ks + c) ^ DecSwizzle<D>::k(16 * gi + n)) * 16);
        const int row = 16 * gi + 4 * c + (n >> 2);
        t_off[gi] = row * (D * 2) + (n & 1) * 8;
        t_sw[gi] = DecSwizzle<D>::v(row);
    }

    df32x4_t acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = df32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, lsum = 0.f;               // maximum of head n; this lane's part of its sum
    DFrag qf[KS];
    int q_rot = -1;
    const int nh = n % MAXG, np = n / MAXG;        // head of this lane; which of the P tiles in a register is its own
    df32x4_t held[R][2];                           // logits of the tiles since the last stores
    int done = 0;
    float* lbase = logits + ((size_t)bh * n_tiles + np * W) * (kDecRows * MAXG) + (nh * 4 + c) * 4;
#pragma nounroll                                   // (nor peeled: a second copy of the loop is fetched with a cold cache)
    while (cons.tile < t_end) {
        const bool in_spare = has_spare && done == DEPTH;
        const int stage = DEPTH == 1 ? 0 : done & (DEPTH - 1);
        static_assert(DEPTH == 1 || DEPTH == 2, "the counts below");
        // tiles behind this one that are on their way, and whether one follows that is to take this one's stage
        const bool next1 = DEPTH == 2 ? cons.tile + W < t_end : has_spare && done == 0, more = cons.tile + DEPTH * W < t_end && !(kSpare && has_spare);
        if (cons.rot != q_rot) {
            // B operand: the group's queries turned by (own index) - (cache index - slot index) of the run
            // (the stored keys are rotated to their slot index), scaled, as bf16.  (Past the first tile the wait for
            // the (cos, sin) loads also waits for the copies in flight: once per run.)
            q_rot = cons.rot;
            if (done == 0) { if (next1) wait_vm_fenced<4 * NC>(); else wait_vm_fenced<2 * NC>(); }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[ks].u = du32x4_t{0u, 0u, 0u, 0u};
            if (nh < g.G) {
                float4 w[KS / 2][4];               // (cos, sin) of 8 rotary pairs per step
                if (done == 0) {
                    const float* cs = reinterpret_cast<const float*>(&csbuf[wave][0]);
#pragma unroll
                    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
                        for (int x = 0; x < 4; ++x) w[ks][x] = *reinterpret_cast<const float4*>(cs + (ks * 32 + c * 8 + 2 * x) * 2);
                } else {
                    const float2* cs = rope + (size_t)q_rot * (D / 2);
#pragma unroll
                    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
                        for (int x = 0; x < 4; ++x) w[ks][x] = *reinterpret_cast<const float4*>(cs + ks * 32 + c * 8 + 2 * x);
                }
                const bf16_t* qh = reinterpret_cast<const bf16_t*>(&qbuf[wave][0]) + nh * D;
#pragma unroll
                for (int ks = 0; ks < KS / 2; ++ks) {
                    const int e = ks * 32 + c * 8;
                    float x0[8], x1[8], y0[8], y1[8];
                    Vec8<bf16_t>::load(qh + e, x0);
                    Vec8<bf16_t>::load(qh + e + D / 2, x1);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float cw = i & 1 ? w[ks][i >> 1].z : w[ks][i >> 1].x, sw = i & 1 ? w[ks][i >> 1].w : w[ks][i >> 1].y;
                        y0[i] = rot_lo(x0[i], x1[i], cw, sw) * qscale;
                        y1[i] = rot_hi(x0[i], x1[i], cw, sw) * qscale;
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        qf[ks].u[x] = dec_pack_bf16(y0[2 * x], y0[2 * x + 1]);
                        qf[ks + KS / 2].u[x] = dec_pack_bf16(y1[2 * x], y1[2 * x + 1]);
                    }
                }
            }
        }
        // K of this tile has landed.  Issued after it: V of this tile, K and V of the tiles on their way, and (while
        // these are the copies that were on their way then) the stores.  Counting fewer than are outstanding only waits longer.
        const bool stored = done >= HOLD && done % HOLD < DEPTH;
        if (stored) { if (next1) wait_vm_fenced<3 * NC + NS>(); else wait_vm_fenced<NC + NS>(); }
        else        { if (next1) wait_vm_fenced<3 * NC>(); else wait_vm_fenced<NC>(); }
        const unsigned char* kp = in_spare ? &spare[0][0] : ring_w + 2 * stage * kStage;
        // (all fragments of a product are read before it starts: read two ahead, as the compiler would, a tile takes twice as long)
        DFrag kf[2][KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int gi = 0; gi < 2; ++gi) kf[gi][ks].u = *reinterpret_cast<const du32x4_t*>(kp + a_off[gi][ks]);
        wait_lds_reads();                          // the stage may be overwritten now
        __builtin_amdgcn_sched_barrier(0);
        df32x4_t s[2] = {df32x4_t{0.f, 0.f, 0.f, 0.f}, df32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int gi = 0; gi < 2; ++gi) s[gi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[gi][ks].v, qf[ks].v, s[gi], 0, 0, 0);
        if (more) issue(kbh, k_off, prod, ring_lds + 2 * stage * kStage);
        // The logits wait in registers (every column group has the products of all heads) and leave together: all NS stores of
        // HOLD tiles, or, behind the last tile, those that there are (two at least).
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (done / P % R == r && done % P == np) { held[r][0] = s[0]; held[r][1] = s[1]; }
        const bool full = done % HOLD == HOLD - 1;
        if (full || cons.tile + W >= t_end) {
            float* lt = lbase + (ptrdiff_t)(cons.tile - done % HOLD * W) * (kDecRows * MAXG);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r * P <= done % HOLD && r * P + np <= done % HOLD)
#pragma unroll
                    for (int gi = 0; gi < 2; ++gi) {
                        float* to = lt + r * P * W * (kDecRows * MAXG) + gi * (16 * MAXG);
                        if (kThrough) store_16_through(to, held[r][gi]); else *reinterpret_cast<df32x4_t*>(to) = held[r][gi];
                    }
        }
        if (cons.nvalid < kDecRows) {
#pragma unroll
            for (int gi = 0; gi < 2; ++gi)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (16 * gi + 4 * c + j >= cons.nvalid) s[gi][j] = -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
        mx = max_groups(mx);
        if (__any(mx > m + kDecRescale)) {         // (the first tile: m is -infinity)
            const float mn = fmaxf(m, mx), alpha = rescale_of(m, mn);
            m = mn;
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[db][j] *= alpha;
        }
        DFrag pf;
        const float mr = finite_max(m);
#pragma unroll
        for (int gi = 0; gi < 2; ++gi)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const float p0 = __builtin_amdgcn_exp2f(s[gi][2 * x] - mr), p1 = __builtin_amdgcn_exp2f(s[gi][2 * x + 1] - mr);
                lsum += p0 + p1;
                pf.u[2 * gi + x] = dec_pack_bf16(p0, p1);
            }
        // V of this tile has landed.  Issued after it: K and V of the tiles on their way, K of the one that takes this stage, the
        // stores of the last DEPTH tiles and this one
        if (done + 1 >= HOLD && (done + 1) % HOLD < DEPTH) {
            if (more) wait_vm_fenced<(2 * DEPTH - 1) * NC + NS>(); else if (next1) wait_vm_fenced<2 * NC + NS>(); else wait_vm_fenced<NS>();
        } else {
            if (more) wait_vm_fenced<(2 * DEPTH - 1) * NC>(); else if (next1) wait_vm_fenced<2 * NC>(); else wait_vm_fenced<2>();
        }
        const unsigned char* vp = in_spare ? &spare[kSpare ? 1 : 0][0] : ring_w + (2 * stage + 1) * kStage;
        DFrag vf[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const uint2 r = read_tr16(vp + t_off[hf] + (((2 * db + ((n & 3) >> 1)) ^ t_sw[hf]) * 16));
                vf[db].u[2 * hf] = r.x;
                vf[db].u[2 * hf + 1] = r.y;
            }
        wait_lds_reads();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[db].v, pf.v, acc[db], 0, 0, 0);
        if (more) {
            issue(vbh, v_off, prod, ring_lds + (2 * stage + 1) * kStage);
            prod.advance(lr, W);
        }
        ++done;
        cons.advance(lr, W);
    }
    if (split == 0) own.finish(g, b, hk, qscale, part, n_splits);
    lsum = sum_groups(lsum);
    // The waves' results meet in LDS once: every wave leaves its sums as they are in its own ring (nothing is on its way there
    // any more), and whoever adds them up scales them to the common maximum.
    if (c == 0) red[n][wave] = make_float2(m, lsum);
    float* osum = reinterpret_cast<float*>(&ring[wave][0][0][0]);   // [MAXG][D]: this lane holds, for head n, elements 16*db + 4*c + j
    if (n < MAXG)
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<df32x4_t*>(&osum[n * D + 16 * db + 4 * c]) = acc[db];
    __syncthreads();
    for (int idx = threadIdx.x; idx < g.G * D; idx += kAttendThreads) {
        const int hh = idx / D;
        float2 ml[W];
        float x[W], mm = -INFINITY, s = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) { ml[w] = red[hh][w]; x[w] = reinterpret_cast<const float*>(&ring[w][0][0][0])[idx]; }
#pragma unroll
        for (int w = 0; w < W; ++w) mm = fmaxf(mm, ml[w].x);
#pragma unroll
        for (int w = 0; w < W; ++w)                // (a wave without tiles adds nothing; NaN stays NaN)
            s += x[w] * (ml[w].y > 0.f ? __builtin_amdgcn_exp2f(ml[w].x - mm) : ml[w].x == -INFINITY ? 0.f : ml[w].y);
        opart[(((size_t)b * g.Hq + hk * g.G + hh) * n_splits + split) * D + idx % D] = s;
    }
    if (wave == W - 1 && l < g.G) {
        float mm = -INFINITY, ll = 0.f;
        for (int w = 0; w < W; ++w) ml_merge(mm, ll, red[l][w].x, red[l][w].y);
        float* p = part_of(part, (size_t)b * g.Hq + hk * g.G + l, n_splits, split);
        p[0] = mm;
        p[1] = ll;
    }
}

// ------------------------------------------------------------------ attend, fp32: VALU
//
// The same split results in fp32 arithmetic.  Sixteen lanes share a row, every lane owns D/16 contiguous
// elements of it and all heads of the group; a workgroup takes four tiles (128 rows) at a time, eight
// consecutive rows per lane group, all eight loads of K and of V in flight together.  Bound by the latency of one
// round where the cache is small, by the products in the lanes where it is large; from 3 heads a group at d = 128 on a
// SIMD holds one wave (256 registers).  8 heads of 4K slots, us a step with separate passes over K and V and
// with this: d = 64, groups of 4 heads 59.2 -> 31.8; d = 128, groups of 1, 4 and 8 42.0 -> 21.9, 78.3 -> 46.8,
// 131.7 -> 83.5.
template <int D, int MAXG>
__global__ __launch_bounds__(kDecThreads) void decode_attend_f32_kernel(
    Geom g, DecodeRuns runs, Splits sp, float qscale, const float* __restrict__ q, const float* __restrict__ k_new,
    const float* __restrict__ Kr, const float* __restrict__ Vc, const float2* __restrict__ rope, float* __restrict__ logits,
    float* __restrict__ part, float* __restrict__ opart)
{
    constexpr int EPL = D / 16, U = 8, kTiles = 4;
    __shared__ float ps[kTiles * kDecRows][MAXG];          // logits, then probabilities of the 128 rows
    __shared__ float alpha_s[MAXG];
    __shared__ float osum[kDecWaves][MAXG][D];
    const int n_tiles = runs.n_tiles, n_splits = sp.n;
    const int split = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
    const int bh = b * g.Hkv + hk;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int lane = threadIdx.x % 16, r0 = (threadIdx.x % 64 / 16) * U;   // wave w takes tile w of the four, a lane group rows r0 .. r0 + 7 of it
    const int t_first = split * sp.each + min(split, sp.more), t_end = t_first + sp.each + (split < sp.more ? 1 : 0);
    if (split == 0) {
        OwnLogits<float, D, kDecWaves> own;
        own.load(g, b, hk, q, k_new);
        own.finish(g, b, hk, qscale, part, n_splits);
    }
    float o[MAXG][EPL], qr[MAXG][EPL];
#pragma unroll
    for (int hh = 0; hh < MAXG; ++hh)
#pragma unroll
        for (int x = 0; x < EPL; ++x) { o[hh][x] = 0.f; qr[hh][x] = 0.f; }
    float m_run[(MAXG + kDecWaves - 1) / kDecWaves], l_run[(MAXG + kDecWaves - 1) / kDecWaves];   // heads wave, wave + 4
#pragma unroll
    for (int i = 0; i < (MAXG + kDecWaves - 1) / kDecWaves; ++i) { m_run[i] = -INFINITY; l_run[i] = 0.f; }
    TileWalk t;
    t.seek(LaneRuns(runs), t_first + wave);
    int q_rot = -1;
    for (int tb = t_first; tb < t_end; tb += kTiles, t.advance(runs, kTiles)) {
        const bool have = t.tile < t_end;
        float vv[U][EPL];
        if (have) {
            if (t.rot != q_rot) {
                q_rot = t.rot;
                const float2* cs = rope + (size_t)q_rot * (D / 2);
#pragma unroll
                for (int hh = 0; hh < MAXG; ++hh)
                    if (hh < g.G) {
                        const float* qh = q + ((size_t)b * g.Hq + hk * g.G + hh) * D;
#pragma unroll
                        for (int x = 0; x < EPL; ++x) {
                            const int e = lane * EPL + x, pe = e < D / 2 ? e : e - D / 2;
                            const float2 w = cs[pe];
                            qr[hh][x] = (e < D / 2 ? rot_lo(qh[pe], qh[pe + D / 2], w.x, w.y) : rot_hi(qh[pe], qh[pe + D / 2], w.x, w.y)) * qscale;
                        }
                    }
            }
            const size_t row0 = (size_t)bh * g.slots + t.start;
            float kv[U][EPL];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t off = (row0 + min(r0 + u, t.nvalid - 1)) * D + lane * EPL;
#pragma unroll
                for (int x = 0; x < EPL; x += 4) {
                    *reinterpret_cast<float4*>(&kv[u][x]) = *reinterpret_cast<const float4*>(Kr + off + x);
                    *reinterpret_cast<float4*>(&vv[u][x]) = *reinterpret_cast<const float4*>(Vc + off + x);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int hh = 0; hh < MAXG; ++hh) {
                    float a = 0.f;
#pragma unroll
                    for (int x = 0; x < EPL; ++x) a += qr[hh][x] * kv[u][x];
#pragma unroll
                    for (int w = 8; w > 0; w >>= 1) a += __shfl_xor(a, w, 16);
                    if (lane == 0) {
                        ps[wave * kDecRows + r0 + u][hh] = r0 + u < t.nvalid ? a : -INFINITY;
                        logits[((size_t)bh * n_tiles + t.tile) * (kDecRows * MAXG) + logit_index<MAXG>(r0 + u, hh)] = a;
                    }
                }
        } else if (lane == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int hh = 0; hh < MAXG; ++hh) ps[wave * kDecRows + r0 + u][hh] = -INFINITY;
        }
        __syncthreads();
        // wave w: the 128 rows of heads w and w + 4
#pragma unroll
        for (int i = 0; i < (MAXG + kDecWaves - 1) / kDecWaves; ++i) {
            const int hh = wave + i * kDecWaves;
            if (hh < g.G) {
                const float a0 = ps[l][hh], a1 = ps[l + 64][hh];
                float mx = fmaxf(a0, a1);
#pragma unroll
                for (int w = 32; w > 0; w >>= 1) mx = fmaxf(mx, __shfl_xor(mx, w, 64));
                const float mn = fmaxf(m_run[i], mx), mr = finite_max(mn), alpha = rescale_of(m_run[i], mn), p0 = exp2f(a0 - mr), p1 = exp2f(a1 - mr);
                float sum = p0 + p1;
#pragma unroll
                for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
                m_run[i] = mn;
                l_run[i] = l_run[i] * alpha + sum;
                ps[l][hh] = p0;
                ps[l + 64][hh] = p1;
                if (l == 0) alpha_s[hh] = alpha;
            }
        }
        __syncthreads();
#pragma unroll
        for (int hh = 0; hh < MAXG; ++hh)
            if (hh < g.G) {
                const float alpha = alpha_s[hh];
#pragma unroll
                for (int x = 0; x < EPL; ++x) o[hh][x] *= alpha;
                if (have && r0 < t.nvalid) {       // (a lane group without rows would add zero times the last row)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float p = ps[wave * kDecRows + r0 + u][hh];
#pragma unroll
                        for (int x = 0; x < EPL; ++x) o[hh][x] += p * vv[u][x];
                    }
                }
            }
        __syncthreads();
    }
    // the four lane groups of a wave add up through lane shuffles, the waves through LDS
#pragma unroll
    for (int hh = 0; hh < MAXG; ++hh)
#pragma unroll
        for (int x = 0; x < EPL; ++x) {
            float s = o[hh][x];
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (l < 16) osum[wave][hh][lane * EPL + x] = s;
        }
#pragma unroll
    for (int i = 0; i < (MAXG + kDecWaves - 1) / kDecWaves; ++i) {
        const int hh = wave + i * kDecWaves;
        if (hh < g.G && l == 0) {
            float* p = part_of(part, (size_t)b * g.Hq + hk * g.G + hh, n_splits, split);
            p[0] = m_run[i];
            p[1] = l_run[i];
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < g.G * D; idx += kDecThreads) {
        const int hh = idx / D, e = idx % D;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kDecWaves; ++w) s += osum[w][hh][e];
        opart[(((size_t)b * g.Hq + hk * g.G + hh) * n_splits + split) * D + e] = s;
    }
}

// ------------------------------------------------------------------ finish
//
// Workgroups of one (sequence, KV head), told apart by blockIdx.x; none waits for another:
//   0            the token's own score and its insertion (Alg. 2 for one token)
//   1 .. G       the output of one query head: the splits' outputs and the own value, combined
//   the rest     the EMA step of the cached rows' scores
// The insertion reads and replaces at most one cached row per cascade (DecodeInsert names their slots,
// which follow from the structure alone): workgroup 0 takes the EMA step of those rows itself and the
// others leave them out, so the whole step needs no order between workgroups.
// Bound by latency: every workgroup loads what it may need before it waits for the combined maxima, and nothing it
// loads depends on another load but through the arguments: the runs of the step are looked up in registers, and the
// place of the insertion's logits comes from the host.  A workgroup at 8K slots, from its start: insertion 6.2 -> 3.2 us, outputs
// 1.8, scores 2.6.
// parts: what a launch does.  Homogeneous heads share their scores between the EMA step and the
// insertion, and the diagnostic snapshot is taken there: those steps launch the two parts one after the other.
constexpr int kFinishScores = 1, kFinishRest = 2;

__device__ inline float reduce_heads(const Geom& g, float red, float p) { return g.head_reduce == CASCADE_REDUCE_MAX ? fmaxf(red, p) : red + p; }

template <typename T, int D, int MAXG>
__global__ __launch_bounds__(kDecThreads) void decode_finish_kernel(
    Geom g, DecodeRuns runs, DecodeInsert ins, int parts, int n_splits, int tiles_per_wg, int qstride, const float2* __restrict__ rope,
    const float* __restrict__ logits, const float* __restrict__ part, const float* __restrict__ opart, const T* __restrict__ k_new,
    const T* __restrict__ v_new, T* __restrict__ out, T* __restrict__ Kc, T* __restrict__ Kr, T* __restrict__ Vc, float* __restrict__ mu,
    int32_t* __restrict__ ids, int32_t* __restrict__ swaps, float* __restrict__ mu_chunk)
{
    __shared__ float lse_s[MAXG], own_s[MAXG];
    __shared__ float buf[kDecThreads * 4];
    const int role = blockIdx.x + (parts & kFinishRest ? 0 : 1 + g.G), hk = blockIdx.y, b = blockIdx.z;
    const int bh = b * g.Hkv + hk, tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
    const bool both = parts == (kFinishScores | kFinishRest);

    // log2-sum-exp2 of the heads of a group, the own key included: head wave (and wave + 4) by this wave, an entry per lane.
    // The loads are issued first of all.
    constexpr int NH = (MAXG + kDecWaves - 1) / kDecWaves;
    float2 entry[NH];
    float own_logit[NH];
    auto load_entries = [&](int kv_head) {
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const float* p = part + ((size_t)b * g.Hq + kv_head * g.G + min(wave + i * kDecWaves, g.G - 1)) * (n_splits + 1) * 2;
            entry[i] = *reinterpret_cast<const float2*>(p + 2 * min(l, n_splits));
            own_logit[i] = p[2 * n_splits];
        }
    };
    auto combine = [&](int kv_head) {
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const int hh = wave + i * kDecWaves;
            if (hh >= g.G) break;
            const float* p = part + ((size_t)b * g.Hq + kv_head * g.G + hh) * (n_splits + 1) * 2;
            float m = -INFINITY, s = 0.f;
            if (l <= n_splits) ml_merge(m, s, entry[i].x, entry[i].y);
            for (int e = l + 64; e <= n_splits; e += 64) ml_merge(m, s, p[2 * e], p[2 * e + 1]);
            const float mm = wave_max(m);
            s = wave_sum(m == -INFINITY ? 0.f : s * __builtin_amdgcn_exp2f(m - mm));
            if (l == 0) { lse_s[hh] = mm + __log2f(s); own_s[hh] = own_logit[i]; }
        }
        __syncthreads();
    };
    const int n_tiles = runs.n_tiles;
    if (role > 0) load_entries(hk);
    const float beta = g.beta, omb = 1.f - g.beta;

    if (role > g.G) {
        // ---- scores: a thread takes four consecutive rows of a tile (16 gi + 4 c .. + 3)
        const int t0 = (role - 1 - g.G) * tiles_per_wg, t1 = min(n_tiles, t0 + tiles_per_wg);
        const int sub = tid & 7, gi = sub >> 2, c = sub & 3;
        bool first = true;
        const LaneRuns lr(runs);
        for (int tb = t0; tb < t1; tb += kDecThreads / 8) {
            const int tile = tb + tid / 8;
            // the run of the tile: every thread counts the runs that begin at or before it
            int si = 0;
#pragma unroll
            for (int i = 1; i < 16; ++i) si += tile >= runs.tile0[i] ? 1 : 0;
            if (runs.n > 16)
#pragma unroll
                for (int i = 16; i < kMaxDecodeRuns; ++i) si += tile >= runs.tile0[i] ? 1 : 0;
            const int rt = tile - __shfl(lr.tile0, si, 64);
            const int start = __shfl(lr.start, si, 64) + rt * kDecRows, nvalid = min(kDecRows, __shfl(lr.len, si, 64) - rt * kDecRows);
            const int r0 = 16 * gi + 4 * c;
            const bool have = tile < t1 && r0 < nvalid;
            float4 lg[MAXG];
            float old[4];
            float* pm = mu + (size_t)bh * g.slots + start + r0;
            if (have) {
                const float* lt = logits + ((size_t)bh * n_tiles + tile) * (kDecRows * MAXG);
#pragma unroll
                for (int hh = 0; hh < MAXG; ++hh) lg[hh] = *reinterpret_cast<const float4*>(lt + logit_index<MAXG>(r0, hh));
#pragma unroll
                for (int j = 0; j < 4; ++j) old[j] = r0 + j < nvalid ? pm[j] : 0.f;
            }
            int mine = 0;                                  // rows that exist and are not the insertion's (those are workgroup 0's)
#pragma unroll
            for (int j = 0; j < 4; ++j) mine |= r0 + j < nvalid ? 1 << j : 0;
            if (both)
                for (int i = 0; i < ins.n; ++i) {
                    const int r = ins.slot[i] - (start + r0);
                    if (r >= 0 && r < 4) mine &= ~(1 << r);
                }
            if (first) { combine(hk); first = false; }     // (uniform; behind the first loads)
            if (have) {
                float red[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int hh = 0; hh < MAXG; ++hh)
                    if (hh < g.G) {
                        const float lse = lse_s[hh];
                        red[0] = reduce_heads(g, red[0], __builtin_amdgcn_exp2f(lg[hh].x - lse));
                        red[1] = reduce_heads(g, red[1], __builtin_amdgcn_exp2f(lg[hh].y - lse));
                        red[2] = reduce_heads(g, red[2], __builtin_amdgcn_exp2f(lg[hh].z - lse));
                        red[3] = reduce_heads(g, red[3], __builtin_amdgcn_exp2f(lg[hh].w - lse));
                    }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (mine >> j & 1)
                        pm[j] = beta * old[j] + omb * (g.head_reduce == CASCADE_REDUCE_MAX ? red[j] : red[j] / (float)g.G);
            }
        }
        return;
    }

    if (role > 0) {
        // ---- output of query head hk * G + role - 1: four elements per thread, the splits over the thread groups
        constexpr int TPR = D / 4, NG = kDecThreads / TPR;
        const int hh = role - 1, e4 = tid % TPR, sg = tid / TPR;
        const size_t head = (size_t)b * g.Hq + hk * g.G + hh;
        const float* p = part + head * (n_splits + 1) * 2;
        const float4* op = reinterpret_cast<const float4*>(opart + head * n_splits * D) + e4;
        // the first splits' outputs are on their way while the maxima are combined
        constexpr int kEarly = 4;
        float4 x[kEarly];
        float2 ml[kEarly];
#pragma unroll
        for (int i = 0; i < kEarly; ++i) {
            const int s = min(sg + i * NG, n_splits - 1);
            x[i] = op[(size_t)s * TPR];
            ml[i] = *reinterpret_cast<const float2*>(p + 2 * s);
        }
        const float vn = tid < D ? Elem<T>::load(v_new + ((size_t)b * g.Hkv + hk) * D + tid) : 0.f;
        combine(hk);
        const float lse = lse_s[hh];
        auto weight = [&](float m, float l) { return l == 0.f ? 0.f : __builtin_amdgcn_exp2f(m - lse); };   // an empty split has no maximum
        float4 a = {0.f, 0.f, 0.f, 0.f};
        auto add = [&](float w, const float4& y) { a.x += w * y.x; a.y += w * y.y; a.z += w * y.z; a.w += w * y.w; };
#pragma unroll
        for (int i = 0; i < kEarly; ++i)
            if (sg + i * NG < n_splits) add(weight(ml[i].x, ml[i].y), x[i]);
        for (int s = sg + kEarly * NG; s < n_splits; s += NG) add(weight(p[2 * s], p[2 * s + 1]), op[(size_t)s * TPR]);
        reinterpret_cast<float4*>(buf)[tid] = a;
        __syncthreads();
        if (tid < D) {
            float s = __builtin_amdgcn_exp2f(own_s[hh] - lse) * vn;
#pragma unroll
            for (int x = 0; x < NG; ++x) s += buf[x * D + tid];
            Elem<T>::store(out + head * D + tid, s);
        }
        return;
    }

    // ---- the token's score, and its insertion
    // Everything the decisions and the moves may need is loaded first, whatever the decisions will be: the row
    // every cascade may be offered (a thread group per cascade), the scores and logits of the rows that
    // compete or move on (a thread per cascade).
    constexpr int LPR = D / 16;
    const int mine = tid / LPR, lane = tid % LPR;
    const int own_entry = min(tid, kMaxCascades - 1);
    int dst = ins.slot[min(mine, kMaxCascades - 1)], src = ins.slot[min(max(mine - 1, 0), kMaxCascades - 1)];
    int rank_slot = ins.slot[own_entry], rank_row = ins.row[own_entry];
    asm volatile("" : "+v"(dst), "+v"(src), "+v"(rank_slot), "+v"(rank_row));           // one wait for all four, not one in each branch
    load_entries(hk);
    const bool ranked = tid < ins.n && insert_kind(ins, own_entry) != kInsertAppend;    // this thread's cascade ranks its item
    float held = 0.f, lg[MAXG];
    if (ranked) {
        held = mu[(size_t)bh * g.slots + rank_slot];
        if (both) {
            const float* lt = logits + ((size_t)bh * n_tiles + rank_row / kDecRows) * (kDecRows * MAXG) + logit_index<MAXG>(rank_row % kDecRows, 0);
#pragma unroll
            for (int hh = 0; hh < MAXG; ++hh) lg[hh] = lt[logit_index<MAXG>(0, hh)];
        }
    }
    Raw8<T> k0, k1, v0, v1;
    float2 cs[8];                                          // of the destination
    int id = ins.id0;
    if (mine < ins.n) {
        const size_t srow = mine == 0 ? (size_t)b * g.Hkv + hk : (size_t)bh * g.slots + src;
        const T *ks = (mine == 0 ? k_new : (const T*)Kc) + srow * D, *vs = (mine == 0 ? v_new : (const T*)Vc) + srow * D;
        if (mine > 0) id = ids[srow];
        k0.load(ks + lane * 8);
        k1.load(ks + D / 2 + lane * 8);
        v0.load(vs + lane * 8);
        v1.load(vs + D / 2 + lane * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) cs[i] = rope[(size_t)dst * (D / 2) + lane * 8 + i];
    }
    // independent heads: the query heads of this KV head; homogeneous heads: all query heads (every
    // workgroup of the sequence computes the same value, group by group in the same order)
    const bool all = g.head_policy == CASCADE_HEADS_HOMOGENEOUS;
    float own = 0.f;
    for (int kv = all ? 0 : hk; kv < (all ? g.Hkv : hk + 1); ++kv) {
        if (all) {                                         // (the previous group's values have been read)
            __syncthreads();
            load_entries(kv);
        }
        combine(kv);
        float red = 0.f;
        for (int hh = 0; hh < g.G; ++hh) red = reduce_heads(g, red, __builtin_amdgcn_exp2f(own_s[hh] - lse_s[hh]));
        if (g.head_reduce == CASCADE_REDUCE_MEAN) red /= (float)g.G;
        own = reduce_heads(g, own, red);
    }
    if (all && g.head_reduce == CASCADE_REDUCE_MEAN) own /= (float)g.Hkv;
    own *= omb;
    if (ranked) {
        if (both) {                                        // (never with homogeneous heads of several KV heads: lse_s is this group's)
            float red = 0.f;
#pragma unroll
            for (int hh = 0; hh < MAXG; ++hh)
                if (hh < g.G) red = reduce_heads(g, red, __builtin_amdgcn_exp2f(lg[hh] - lse_s[hh]));
            held = beta * held + omb * (g.head_reduce == CASCADE_REDUCE_MAX ? red : red / (float)g.G);
        }
        buf[tid] = held;
    }
    __syncthreads();                                       // (every source row has been read, too)
    // Who ends up where: the token (or what the cascade before evicted) is offered to one cascade after the
    // other; it is appended, or takes the place of the oldest item, which moves on, or competes with the
    // newest item, which stays unless the offer's score is strictly higher.
    float offered = own, my_score = 0.f;
    bool my_move = false;
    for (int i = 0; i < ins.n; ++i) {
        const float there = buf[i];
        const bool compete = insert_kind(ins, i) == kInsertCompete, takes = !compete || (g.token_selection && offered > there);
        if (i == mine) { my_move = takes; my_score = takes ? offered : there; }
        if (takes && compete && tid == 0) atomicAdd(&swaps[bh * g.N + i], 1);
        offered = there;
    }
    if (tid == 0) mu_chunk[(size_t)bh * qstride] = own;
    if (mine < ins.n) {
        const size_t drow = (size_t)bh * g.slots + dst;
        if (lane == 0) mu[drow] = my_score;
        if (my_move) {
            k0.store(Kc + drow * D + lane * 8);
            k1.store(Kc + drow * D + D / 2 + lane * 8);
            float x0[8], x1[8];
            k0.values(x0);
            k1.values(x1);
            rotate8<T>(x0, x1, cs, Kr + drow * D + lane * 8, Kr + drow * D + D / 2 + lane * 8);
            v0.store(Vc + drow * D + lane * 8);
            v1.store(Vc + drow * D + D / 2 + lane * 8);
            if (lane == 0) ids[drow] = id;
        }
    }
}

// ------------------------------------------------------------------ launchers

bool decode_supported(const Geom& g) { return (g.d == 64 || g.d == 128) && g.G <= kMaxG; }

int decode_logit_heads(const Geom& g) { return g.G <= 1 ? 1 : (g.G <= 2 ? 2 : (g.G <= 4 ? 4 : 8)); }

int decode_max_tiles(const Geom& g) { return g.slots / kDecRows + 2 * g.N + 1; }

// Where the rows that the insertion ranks lie among the logits.
static DecodeInsert placed(const DecodeInsert& ins, const DecodeRuns& r)
{
    DecodeInsert p = ins;
    for (int i = 0; i < p.n; ++i)
        for (int si = 0; si < r.n; ++si) {
            const int row = p.slot[i] - r.start[si];
            if (row >= 0 && row < r.len[si]) p.row[i] = r.tile0[si] * kDecRows + row;
        }
    return p;
}

static DecodeRuns decode_runs(const SegList& sl)
{
    DecodeRuns r = {};
    r.n = sl.n;
    for (int i = 0; i < kMaxDecodeRuns; ++i) r.tile0[i] = INT32_MAX;
    for (int i = 0; i < sl.n; ++i) {
        r.tile0[i] = r.n_tiles;
        r.start[i] = sl.s[i].start;
        r.len[i] = sl.s[i].len;
        r.rot[i] = sl.qrot0[sl.s[i].qvar];
        r.n_tiles += (sl.s[i].len + kDecRows - 1) / kDecRows;
    }
    return r;
}

int decode_tiles(const SegList& sl)
{
    int n = 0;
    for (int i = 0; i < sl.n; ++i) n += (sl.s[i].len + kDecRows - 1) / kDecRows;
    return n;
}

#define CKV_DECODE_G(fn, T, D)                                 \
    switch (decode_logit_heads(g)) {                           \
        case 1: fn(T, D, 1); break;                            \
        case 2: fn(T, D, 2); break;                            \
        case 4: fn(T, D, 4); break;                            \
        default: fn(T, D, 8); break;                           \
    }

void launch_decode_attend(const Geom& g, int dtype, const DevBuffers& b, const SegList& sl, int n_splits, const void* q, const void* k,
                          hipStream_t s)
{
    const dim3 grid(n_splits, g.Hkv, g.B), block(kDecThreads);
    const DecodeRuns runs = decode_runs(sl);
    const Splits sp = {n_splits, runs.n_tiles / n_splits, runs.n_tiles % n_splits};
    const float qscale = g.scale * kLog2e;
#define CKV_ATTEND_F32(T, D, MG)                                                                                          \
    hipLaunchKernelGGL((decode_attend_f32_kernel<D, MG>), grid, block, 0, s, g, runs, sp, qscale, (const T*)q, \
                       (const T*)k, (const T*)b.Kr, (const T*)b.Vc, b.rope, b.logits, b.part, b.opart)
    // Eight registers' worth of logits are held where some wave has more tiles than fit in one; both sides are measured at
    // decode_attend_kernel
    const bool hold = sp.each + (sp.more > 0) > kAttendWaves * (16 / decode_logit_heads(g));
#define CKV_ATTEND_MFMA_R(T, D, MG, R)                                                                                    \
    hipLaunchKernelGGL((decode_attend_kernel<D, MG, R>), grid, dim3(kAttendThreads), 0, s, g, runs, sp, qscale, (const T*)q,  \
                       (const T*)k, (const T*)b.Kr, (const T*)b.Vc, b.rope, b.logits, b.part, b.opart)
#define CKV_ATTEND_MFMA(T, D, MG) if (hold) CKV_ATTEND_MFMA_R(T, D, MG, 8); else CKV_ATTEND_MFMA_R(T, D, MG, 1)
    if (dtype == CASCADE_F32) {
        if (g.d == 128) { CKV_DECODE_G(CKV_ATTEND_F32, float, 128) } else { CKV_DECODE_G(CKV_ATTEND_F32, float, 64) }
    } else {
        if (g.d == 128) { CKV_DECODE_G(CKV_ATTEND_MFMA, bf16_t, 128) } else { CKV_DECODE_G(CKV_ATTEND_MFMA, bf16_t, 64) }
    }
#undef CKV_ATTEND_F32
#undef CKV_ATTEND_MFMA
#undef CKV_ATTEND_MFMA_R
}

void launch_decode_finish(const Geom& g, int dtype, const DevBuffers& b, const SegList& sl, const DecodeInsert& ins, int n_splits, bool scores,
                          bool rest, int qstride, const void* k, const void* v, void* out, hipStream_t s)
{
    const DecodeRuns runs = decode_runs(sl);
    const DecodeInsert at = placed(ins, runs);
    const int n_tiles = runs.n_tiles;
    // score workgroups: 32 tiles each (one round of their threads), up to four rounds where there are many
    int per_wg = 32;
    while (per_wg < 128 && (long)g.B * g.Hkv * ((n_tiles + per_wg - 1) / per_wg) > 2048) per_wg *= 2;
    const int wgs = (rest ? 1 + g.G : 0) + (scores ? (n_tiles + per_wg - 1) / per_wg : 0);
    if (wgs == 0) return;
    const dim3 grid(wgs, g.Hkv, g.B), block(kDecThreads);
    const int parts = (scores ? kFinishScores : 0) | (rest ? kFinishRest : 0);
#define CKV_FINISH(T, D, MG)                                                                                                       \
    hipLaunchKernelGGL((decode_finish_kernel<T, D, MG>), grid, block, 0, s, g, runs, at, parts, n_splits, per_wg, qstride, b.rope, \
                       b.logits, b.part, b.opart, (const T*)k, (const T*)v, (T*)out, (T*)b.Kc, (T*)b.Kr, (T*)b.Vc, b.mu, b.ids,     \
                       b.swaps, b.mu_chunk)
    if (dtype == CASCADE_F32) {
        if (g.d == 128) { CKV_DECODE_G(CKV_FINISH, float, 128) } else { CKV_DECODE_G(CKV_FINISH, float, 64) }
    } else {
        if (g.d == 128) { CKV_DECODE_G(CKV_FINISH, bf16_t, 128) } else { CKV_DECODE_G(CKV_FINISH, bf16_t, 64) }
    }
#undef CKV_FINISH
}

}  // namespace ckv
