// bf16 MFMA kernel of the exact EMA score sums of a chunk (Section 3.1, coefficients of Alg. 3).
//
// MFMA used: v_mfma_f32_32x32x16_bf16, D[m][n] += sum_k A[m][k] B[k][n] with, for lane l,
//   A: row m = l%32, k = 8*(l/32) .. +7        B: column n = l%32, k = 8*(l/32) .. +7
//   D: column n = l%32, rows 8*(j/4) + 4*(l/32) + j%4 for accumulator register j = 0..15.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>

#include "async_copy.h"
#include "mfma_util.h"

namespace ckv {

// ------------------------------------------------------------------ exact score sums

// Key-stationary: a wave keeps 64 keys (two 32-key blocks) in registers as the B operand and
// runs the last `tail` query rows of every head of the group past them (S = Q K^T, one lane owns
// one key column per block).  With the stored log-sum-exp the probabilities are exact:
// p = 2^(s - t[row]) (the queries carry the softmax scale and log2 e) with
// t = lse*log2(e) - log2(weight of the row).  Column sums are an in-lane sum plus one exchange
// with lane l^32; no atomics, so results are identical from run to run.
//
// The query rows reach LDS by asynchronous copies through a ring of three 64-row stages shared
// by the workgroup (one barrier per stage, the copies of the next two stages in flight while a
// stage is used; three workgroups per CU), running on across the heads of the group, so no wave
// waits for a staging round trip.  The exponent offsets come from a small table
// negt[head][row] = -t (-inf for rows that do not contribute, and for the padding behind the
// chunk), written by the attention kernel when it finishes a row; the accumulators start from
// it: a probability is then one v_exp_f32 of an accumulator.
constexpr int kScoreThreads = 256;
constexpr int kScoreKeysPerBlock = 128;   // keys per workgroup and key block of its waves (4 waves x 32)
constexpr int kStStages = 3;
constexpr int kStRows = kScorePadRows;

template <int D> struct ScoreSwz {   // permutation of the 16-byte pieces of a staged row
    __device__ static int of(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
};

// The segments cut into blocks of the keys a workgroup takes: first block of every segment (INT32_MAX behind the last).
struct KeyBlocks {
    int total;
    int first[kMaxSegments];
};

// NKB: 32-key blocks per wave.  Two halve the LDS reads per MFMA; one gives twice as many
// workgroups, for launches that would otherwise leave compute units without work.
template <int D, int NKB>
__global__ __launch_bounds__(kScoreThreads, 3) void score_stream_kernel(
    Geom g, SegList sl, KeyBlocks kbs, int Q, int qstride, int tail, int qpad, int row_parts, float decay, const bf16_t* __restrict__ Qr,
    const bf16_t* __restrict__ Kr, const bf16_t* __restrict__ Krc, const float* __restrict__ negt,
    float* __restrict__ mu, float* __restrict__ mu_chunk, float* __restrict__ sums)
{
    constexpr int KS = D / 16;
    constexpr int kScoreKeys = kScoreKeysPerBlock * NKB, kWaveKeys = 32 * NKB;
    constexpr int PPR = D / 8;                       // 16-byte pieces per row
    constexpr int RPI = 64 / PPR;                    // rows per copy instruction
    constexpr int kStageBytes = kStRows * D * 2;
    constexpr int NCW = kStageBytes / 1024 / 4;      // row copies per wave and stage
    constexpr int NOPS = NCW + 1;                    // vector memory operations per wave and stage
    __shared__ __attribute__((aligned(1024))) unsigned char ring[kStStages][kStageBytes];
    __shared__ __attribute__((aligned(256))) float tneg[kStStages][4][kStRows];   // every wave keeps its own copy
    const int BH = g.B * g.Hkv, n_tiles = kbs.total;
    const int bh = blockIdx.x % BH;
    const int list_tile = (blockIdx.x / BH) % n_tiles, part = blockIdx.x / BH / n_tiles;
    const int b = bh / g.Hkv, hk = bh % g.Hkv;
    const int si = table_entry(kbs.first, list_tile), tile = list_tile - kbs.first[si];
    const Seg sg = sl.s[si];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l32 = l & 31, half = l >> 5;
    const int wave_k0 = tile * kScoreKeys + wave * kWaveKeys;   // first key of this wave inside the segment

    // this wave's keys as B operands (rows past the end of the segment repeat its last row)
    Frag kf[NKB][KS];
    int kk[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        kk[kb] = wave_k0 + kb * 32 + l32;
        const int kc = min(kk[kb], sg.len - 1);
        const bf16_t* krow = sg.chunk ? Krc + ((size_t)bh * Q + kc) * D : Kr + ((size_t)bh * g.slots + sg.start + kc) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[kb][ks].u = *reinterpret_cast<const u32x4_t*>(krow + ks * 16 + half * 8);
    }
    // fragment reads of this lane: row block rb, step ks: row 32*rb + l32, piece 2*ks + half (rows 32 apart are
    // permuted alike)
    int a_off[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a_off[ks] = l32 * (D * 2) + (((2 * ks + half) ^ ScoreSwz<D>::of(l32)) * 16);

    // This workgroup's heads, and its stages of 64 rows of each: all of both, or one part of one head
    const int head0 = row_parts ? part / row_parts : 0, n_heads = row_parts ? 1 : g.G;
    const int all_stages = (tail + kStRows - 1) / kStRows;
    int st0 = 0, st1 = all_stages;
    if (row_parts) {
        st0 = all_stages * (part % row_parts) / row_parts;
        st1 = all_stages * (part % row_parts + 1) / row_parts;
    }
    if (sg.chunk) st0 = max(st0, (tile * kScoreKeys - (Q - tail)) / kStRows);   // earlier rows see none of these keys
    const int i_first = Q - tail + st0 * kStRows;              // first row that contributes
    const int spp = max(st1 - st0, 0);                         // stages per head
    const int T = n_heads * spp;
    const uint32_t ring_lds = lds_address(&ring[0][0]), tneg_lds = lds_address(&tneg[0][0][0]);
    // the keys are in registers before the first copy is issued (a wait for them inside the loop
    // would also wait for every copy in flight)
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[kb][ks].u));
    // what a lane copies of a stage: row x*RPI + l/PPR of the stage, one 16-byte piece (lane constants)
    uint32_t copy_off[NCW];
#pragma unroll
    for (int y = 0; y < NCW; ++y) {
        const int row = (wave * NCW + y) * RPI + l / PPR;
        copy_off[y] = (uint32_t)((row * PPR + ((l % PPR) ^ ScoreSwz<D>::of(row))) * 16);
    }
    int iss_hh = 0, iss_sp = 0;                                 // stage s, the next to issue, is stage iss_sp of head iss_hh
    auto issue = [&](int s) {
        const int i_base = i_first + iss_sp * kStRows;
        const int h = hk * g.G + head0 + iss_hh, slot = s % kStStages;
        if (++iss_sp == spp) { iss_sp = 0; ++iss_hh; }
        const bf16_t* qbase = Qr + (((size_t)sg.qvar * g.B + b) * g.Hq + h) * (size_t)Q * D;
        if (i_base + kStRows <= Q) {          // all rows of the stage exist: the lane offsets are constants
#pragma unroll
            for (int y = 0; y < NCW; ++y)
                async_copy_1k(qbase + (size_t)i_base * D, copy_off[y],
                              __builtin_amdgcn_readfirstlane(ring_lds + slot * kStageBytes + (wave * NCW + y) * 1024));
        } else {
#pragma unroll
            for (int y = 0; y < NCW; ++y) {
                const int x = wave * NCW + y;
                const int row = x * RPI + l / PPR;
                const int piece = (l % PPR) ^ ScoreSwz<D>::of(row);
                async_copy_1k(qbase, (uint32_t)((min(i_base + row, Q - 1) * PPR + piece) * 16),
                              __builtin_amdgcn_readfirstlane(ring_lds + slot * kStageBytes + x * 1024));
            }
        }
        async_copy_256(negt + ((size_t)b * g.Hq + h) * qpad + i_base, (uint32_t)(l * 4),
                       __builtin_amdgcn_readfirstlane(tneg_lds + (uint32_t)((slot * 4 + wave) * kStRows * 4)));
    };

    float red[NKB] = {}, colsum[NKB] = {};
    // A stage whose 64 rows all see all keys of the wave.  Fragments are read kAhead steps before their use and
    // the first MFMAs start from the offsets where they were read: 82 vector and 20 scalar instructions per
    // 32 rows instead of 109 and 65, in a kernel whose exponentials alone are 512 of the vector ALU's cycles
    // per 512 of MFMA: 4096 rows against 16K slots 626 -> 592 us.  (A separate register
    // copy of the offsets or eight steps ahead spill at D = 128; raising the priority of the wave that is ahead
    // in its block changes nothing.)
    auto whole_stage = [&](const unsigned char* qs, const float* tn) {
        constexpr int kAhead = 4;
        static_assert(kAhead <= KS, "the first fragments belong to the first row block");
        Frag fr[kAhead];
        f32x16_t acc[NKB];   // acc[NKB - 1] takes the exponent offsets; the first MFMAs start from there
        auto read_t = [&](int rb) {
#pragma unroll
            for (int jq = 0; jq < 4; ++jq) {
                const float4 t4 = *reinterpret_cast<const float4*>(tn + rb * 32 + jq * 8 + half * 4);
                acc[NKB - 1][jq * 4 + 0] = t4.x; acc[NKB - 1][jq * 4 + 1] = t4.y; acc[NKB - 1][jq * 4 + 2] = t4.z; acc[NKB - 1][jq * 4 + 3] = t4.w;
            }
        };
        auto read_q = [&](int i) { fr[i % kAhead].u = *reinterpret_cast<const u32x4_t*>(qs + a_off[i % KS] + (i / KS) * (64 * D)); };
        read_t(0);
#pragma unroll
        for (int i = 0; i < kAhead; ++i) read_q(i);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[ks % kAhead].v, kf[kb][ks].v, ks == 0 ? acc[NKB - 1] : acc[kb], 0, 0, 0);
                if (rb * KS + ks + kAhead < 2 * KS) read_q(rb * KS + ks + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) colsum[kb] += __builtin_amdgcn_exp2f(acc[kb][j]);
            }
            if (rb == 0) read_t(1);
        }
    };

    int issued = 0;
    for (; issued < kStStages - 1 && issued < T; ++issued) issue(issued);
    int hh = 0, sp = 0;                                         // stage s = stage sp of head hh
    for (int s = 0; s < T; ++s) {
        const int ahead = issued - s - 1;                       // stages issued after stage s
        static_assert(kStStages == 3 || kStStages == 4, "cases below");
        if (kStStages == 4 && ahead >= 2) wait_vm<2 * NOPS>();
        else if (ahead >= 1) wait_vm<NOPS>();
        else wait_vm<0>();
        wg_barrier();    // stage s is complete for every wave, and every wave has left stage s - 1
        if (issued < T) { issue(issued); ++issued; }            // into the slot of stage s - 1
        const int slot = s % kStStages;
        const int i_base = i_first + sp * kStRows;
        const int rows = min(kStRows, Q - i_base);
        const unsigned char* qs = &ring[slot][0];
        if (rows == kStRows && !(sg.chunk && i_base < wave_k0 + kWaveKeys - 1)) whole_stage(qs, &tneg[slot][wave][0]);
        else
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {       // the end of the chunk, the diagonal, rows that see none of the keys
            const int i0 = i_base + rb * 32;
            if (rb * 32 >= rows) continue;
            if (sg.chunk && i0 + 31 < wave_k0) continue;        // chunk keys are seen by later rows only
            f32x16_t acc[NKB];
#pragma unroll
            for (int jq = 0; jq < 4; ++jq) {
                const float4 t4 = *reinterpret_cast<const float4*>(&tneg[slot][wave][rb * 32 + jq * 8 + half * 4]);
                acc[0][jq * 4 + 0] = t4.x; acc[0][jq * 4 + 1] = t4.y; acc[0][jq * 4 + 2] = t4.z; acc[0][jq * 4 + 3] = t4.w;
            }
            if (NKB == 2) acc[NKB - 1] = acc[0];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                Frag qf;
                qf.u = *reinterpret_cast<const u32x4_t*>(qs + a_off[ks] + rb * (64 * D));
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf.v, kf[kb][ks].v, acc[kb], 0, 0, 0);
            }
            if (sg.chunk && i0 < wave_k0 + kWaveKeys - 1) {     // the diagonal crosses this block: mask
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int i = i0 + (j >> 2) * 8 + half * 4 + (j & 3);
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb) {
                        const float p = __builtin_amdgcn_exp2f(acc[kb][j]);
                        colsum[kb] += kk[kb] <= i ? p : 0.f;
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j)
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb) colsum[kb] += __builtin_amdgcn_exp2f(acc[kb][j]);
            }
        }
        if (++sp == spp) {                                      // the head is finished
            sp = 0;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                const float cs = colsum[kb] + __shfl_xor(colsum[kb], 32, 64);
                if (g.head_reduce == CASCADE_REDUCE_MAX) red[kb] = hh == 0 ? cs : fmaxf(red[kb], cs);
                else red[kb] += cs;
                colsum[kb] = 0.f;
            }
            ++hh;
        }
    }
    if (row_parts) {
        // column sums of this part (T == 0: chunk keys that none of its rows sees); score_merge_kernel does the rest
        if (half == 0) {
            float* p = sums + ((size_t)(bh * g.G + head0) * row_parts + part % row_parts) * ((size_t)n_tiles * kScoreKeys) +
                       (size_t)list_tile * kScoreKeys + wave * kWaveKeys + l32;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) p[kb * 32] = red[kb];
        }
        return;
    }
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        float r = red[kb];
        if (g.head_reduce == CASCADE_REDUCE_MEAN) r /= (float)g.G;
        if (half == 0 && kk[kb] < sg.len) {
            if (sg.chunk) mu_chunk[(size_t)bh * qstride + kk[kb]] = r;
            else {
                float* p = mu + (size_t)bh * g.slots + sg.start + kk[kb];
                *p = decay * *p + r;
            }
        }
    }
}

// The parts' column sums of every key added up in a fixed order, the query heads of the group reduced, and the
// EMA step taken (one thread per key).
__global__ __launch_bounds__(2 * kScoreKeysPerBlock) void score_merge_kernel(Geom g, SegList sl, KeyBlocks kbs, int qstride, int row_parts, float decay,
                                                                             const float* __restrict__ sums, float* __restrict__ mu,
                                                                             float* __restrict__ mu_chunk)
{
    const int keys = blockDim.x, bh = blockIdx.y, n_tiles = kbs.total;
    const int si = table_entry(kbs.first, (int)blockIdx.x), tile = (int)blockIdx.x - kbs.first[si];
    const Seg sg = sl.s[si];
    const int k = tile * keys + threadIdx.x;
    if (k >= sg.len) return;
    const size_t stride = (size_t)n_tiles * keys;
    const float* p = sums + (size_t)bh * g.G * row_parts * stride + (size_t)blockIdx.x * keys + threadIdx.x;
    float* m = sg.chunk ? mu_chunk + (size_t)bh * qstride + k : mu + (size_t)bh * g.slots + sg.start + k;
    const float old = sg.chunk ? 0.f : *m;
    float red = 0.f;
    for (int hh = 0; hh < g.G; ++hh) {
        float v = 0.f;
        for (int r = 0; r < row_parts; ++r, p += stride) v += *p;
        red = g.head_reduce == CASCADE_REDUCE_MAX ? (hh == 0 ? v : fmaxf(red, v)) : red + v;
    }
    if (g.head_reduce == CASCADE_REDUCE_MEAN) red /= (float)g.G;
    *m = sg.chunk ? red : decay * old + red;
}

void launch_score_mfma(const Geom& g, const DevBuffers& b, const SegList& sl, int Q, int max_chunk,
                       int tail_rows, float decay, hipStream_t s)
{
    auto tiles_of = [&](int keys) {
        int tiles = 0;
        for (int i = 0; i < sl.n; ++i) tiles += (sl.s[i].len + keys - 1) / keys;
        return tiles;
    };
    const int BH = g.B * g.Hkv, stages = (tail_rows + kStRows - 1) / kStRows;
    const int wide = tiles_of(2 * kScoreKeysPerBlock) * BH;
    // Every head by itself, and in small launches its rows in parts of at least 8 stages: the launch is then spread evenly over the compute
    // units (640 workgroups on 768 slots leave a third of them with two instead of three), for a second launch of
    // 5 to 6 us.  us a call, whole against in parts: 4096 rows against 16K slots 1796 -> 1727, against 2K slots
    // 756 -> 644 in one part a head and 622 in four; 512 rows against 8K slots
    // 158.7 -> 157.0 (against half as many keys a wave); 300 rows, 64 workgroups 36 -> 23
    // for the kernels.  With fewer stages than that the second launch costs more than the balance gives: 264 rows against
    // 16K slots 589 whole, 593 in parts.
    int row_parts = 0;
    if (stages >= 8 || (wide < 256 && stages >= 4)) {
        row_parts = 1;
        while (wide * g.G * row_parts < 1536 && stages / (2 * row_parts) >= 8) row_parts *= 2;
        if (g.G * row_parts == 1) row_parts = 0;
    }
    if (b.opt_score_parts >= 0) row_parts = std::min(b.opt_score_parts, stages);
    // 256 keys per workgroup unless that leaves a good part of the 256 x 3 workgroup slots empty
    bool narrow = row_parts == 0 && wide < 600;
    if (b.opt_score_narrow >= 0) narrow = b.opt_score_narrow == 1;
    const int keys = narrow ? kScoreKeysPerBlock : 2 * kScoreKeysPerBlock, n_tiles = tiles_of(keys);
    // the parts' sums lie where a split attention launch keeps its partial results
    while (row_parts > 0 && (size_t)BH * g.G * row_parts * n_tiles * keys > (size_t)kAttnPartRows * (g.d + 2)) --row_parts;
    KeyBlocks kbs;
    kbs.total = n_tiles;
    for (int i = 0, n = 0; i < kMaxSegments; ++i) {
        kbs.first[i] = i < sl.n ? n : INT32_MAX;
        if (i < sl.n) n += (sl.s[i].len + keys - 1) / keys;
    }
    const dim3 grid(n_tiles * BH * (row_parts ? g.G * row_parts : 1)), block(kScoreThreads);
    const int qpad = max_chunk + kStRows;   // the attention launch left the offsets of this chunk's rows in b.negt
#define CKV_SCORE(D, NKB)                                                                                              \
    hipLaunchKernelGGL((score_stream_kernel<D, NKB>), grid, block, 0, s, g, sl, kbs, Q, max_chunk, tail_rows, qpad, row_parts, decay, \
                       (const bf16_t*)b.Qr, (const bf16_t*)b.Kr, (const bf16_t*)b.Krc, b.negt, b.mu, b.mu_chunk, b.attn_part)
    if (g.d == 128) { if (narrow) CKV_SCORE(128, 1); else CKV_SCORE(128, 2); }
    else { if (narrow) CKV_SCORE(64, 1); else CKV_SCORE(64, 2); }
#undef CKV_SCORE
    if (row_parts)
        hipLaunchKernelGGL(score_merge_kernel, dim3(n_tiles, BH), dim3(keys), 0, s, g, sl, kbs, max_chunk, row_parts, decay, b.attn_part, b.mu,
                           b.mu_chunk);
}

}  // namespace ckv
