// Host-side structure of the cascade update and of the attention segments.
#include "structure.h"

#include <math.h>
#include <string.h>

#include <algorithm>

namespace ckv {

static thread_local std::string g_init_error;
void set_init_error(const std::string& msg) { g_init_error = msg; }
const char* init_error() { return g_init_error.c_str(); }

// ------------------------------------------------------------------ configuration

int check_config(const cascade_config* c, std::string& why)
{
    if (c->batch < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1) { why = "batch and head counts must be positive"; return CASCADE_E_INVALID_CONFIG; }
    if (c->n_q_heads % c->n_kv_heads) { why = "n_q_heads must be a multiple of n_kv_heads"; return CASCADE_E_INVALID_CONFIG; }
    if (c->dtype != CASCADE_F32 && c->dtype != CASCADE_BF16) { why = "dtype must be CASCADE_F32 or CASCADE_BF16"; return CASCADE_E_INVALID_CONFIG; }
    if (c->head_dim < 2 || c->head_dim % 2) { why = "head_dim must be even"; return CASCADE_E_INVALID_CONFIG; }
    if (c->n_sink < 0) { why = "n_sink must not be negative"; return CASCADE_E_INVALID_CONFIG; }
    if (c->n_cascades < 1 || c->n_cascades > CASCADE_MAX_CASCADES) { why = "n_cascades out of range"; return CASCADE_E_INVALID_CONFIG; }
    bool all_zero = true;
    for (int i = 0; i < c->n_cascades; ++i) {
        if (c->cascade_sizes[i] < 1) { why = "every cascade needs at least one slot"; return CASCADE_E_INVALID_CONFIG; }
        if (c->accept_period[i] < 0) { why = "accept_period must not be negative"; return CASCADE_E_INVALID_CONFIG; }
        if (c->accept_period[i] != 0) all_zero = false;
    }
    if (!all_zero) {
        if (c->accept_period[0] != 1) { why = "the first cascade must accept every token (accept_period[0] == 1)"; return CASCADE_E_INVALID_CONFIG; }
        for (int i = 0; i < c->n_cascades; ++i)
            if (c->accept_period[i] < 1) { why = "accept_period entries must be >= 1"; return CASCADE_E_INVALID_CONFIG; }
    }
    if (!(c->ema_beta >= 0.f && c->ema_beta < 1.f)) { why = "ema_beta must be in [0, 1)"; return CASCADE_E_INVALID_CONFIG; }
    if (!(c->rope_base > 0.f)) { why = "rope_base must be positive"; return CASCADE_E_INVALID_CONFIG; }
    if (c->softmax_scale < 0.f) { why = "softmax_scale must not be negative"; return CASCADE_E_INVALID_CONFIG; }
    if (c->max_chunk < 1) { why = "max_chunk must be >= 1"; return CASCADE_E_INVALID_CONFIG; }
    if (c->head_reduce != CASCADE_REDUCE_MAX && c->head_reduce != CASCADE_REDUCE_MEAN) { why = "unknown head_reduce"; return CASCADE_E_INVALID_CONFIG; }
    if (c->token_selection != 0 && c->token_selection != 1) { why = "token_selection must be 0 or 1"; return CASCADE_E_INVALID_CONFIG; }
    if (c->head_policy != CASCADE_HEADS_INDEPENDENT && c->head_policy != CASCADE_HEADS_HOMOGENEOUS) { why = "unknown head_policy"; return CASCADE_E_INVALID_CONFIG; }
    if (c->score_mode != CASCADE_SCORES_EXACT && c->score_mode != CASCADE_SCORES_SINGLE_PASS) { why = "unknown score_mode"; return CASCADE_E_INVALID_CONFIG; }
    if (c->score_mode == CASCADE_SCORES_SINGLE_PASS && c->dtype != CASCADE_BF16) { why = "single-pass scores need dtype CASCADE_BF16"; return CASCADE_E_UNSUPPORTED; }
    long slots = c->n_sink;
    for (int i = 0; i < c->n_cascades; ++i) slots += c->cascade_sizes[i];
    if (slots > (1L << 28)) { why = "cache too large"; return CASCADE_E_INVALID_CONFIG; }
    if (c->dtype == CASCADE_BF16 && c->head_dim != 64 && c->head_dim != 128) { why = "bf16 kernels cover head_dim 64 and 128"; return CASCADE_E_UNSUPPORTED; }
    if (c->dtype == CASCADE_F32 && c->head_dim > 256) { why = "fp32 kernels cover head_dim up to 256"; return CASCADE_E_UNSUPPORTED; }
    return CASCADE_OK;
}

void make_geom(const cascade_config* c, Geom& g)
{
    memset(&g, 0, sizeof(g));
    g.B = c->batch; g.Hq = c->n_q_heads; g.Hkv = c->n_kv_heads; g.G = g.Hq / g.Hkv; g.d = c->head_dim;
    g.n_sink = c->n_sink; g.N = c->n_cascades;
    bool all_zero = true;
    for (int i = 0; i < g.N; ++i) if (c->accept_period[i] != 0) all_zero = false;
    int slots = g.n_sink;
    for (int i = 0; i < g.N; ++i) {
        g.cap[i] = c->cascade_sizes[i];
        g.period[i] = all_zero ? (1 << i) : c->accept_period[i];
        slots += g.cap[i];
    }
    g.slots = slots;
    int base = g.n_sink;                       // physical order: sinks, last cascade, ..., first cascade
    for (int i = g.N - 1; i >= 0; --i) { g.base[i] = base; base += g.cap[i]; }
    g.token_selection = c->token_selection;
    g.head_reduce = c->head_reduce;
    g.head_policy = c->head_policy;
    g.beta = c->ema_beta;
    g.scale = c->softmax_scale > 0.f ? c->softmax_scale : (float)(1.0 / sqrt((double)g.d));
}


static int64_t gcd64(int64_t a, int64_t b)
{
    while (b) { int64_t r = a % b; a = b; b = r; }
    return a;
}

// Alg. 2 applied to Q tokens in order, scores aside.  The items offered to cascade c arrive
// at times tau_k = first + k*step (an arithmetic progression: cascade c-1 only evicts at its
// own accepting times once it is full).  Offer k is
//   APPEND  while the cascade is not full (accepting or eager add),
//   PUSH    when full and tau_k mod period == 0 (the oldest item moves on to cascade c+1),
//   SELECT  when full otherwise (competes with the newest item, one of the two is lost).
void plan_update(const Geom& g, HostState& st, int Q, UpdatePlan& plan)
{
    plan.Q = Q;
    plan.N = g.N;
    plan.sink_fill0 = st.sink_fill;
    plan.n_to_sink = std::min(Q, g.n_sink - st.sink_fill);
    plan.id0 = (int)st.n_seen;
    const int Qc = Q - plan.n_to_sink;

    int64_t first = st.t, step = 1;
    int M = Qc;
    for (int c = 0; c < g.N; ++c) {
        CascStep& cs = plan.c[c];
        const int cap = g.cap[c];
        const int64_t f = g.period[c];
        const bool full0 = st.count[c] == cap;
        cs.cap = cap;
        cs.base = g.base[c];
        cs.M = M;
        cs.A = std::min(M, cap - st.count[c]);
        cs.pstride = (int)(f / gcd64(step, f));
        // offers at accepting times are k = ka + i*pstride for the smallest such ka >= 0
        int ka = -1;
        for (int k = 0; k < cs.pstride && k < M; ++k)
            if ((first + (int64_t)k * step) % f == 0) { ka = k; break; }
        cs.kp0 = M;
        cs.P = 0;
        if (ka >= 0) {
            st.accepted[c] += (M - 1 - ka) / cs.pstride + 1;
            int k = ka;
            if (k < cs.A) k += ((cs.A - k + cs.pstride - 1) / cs.pstride) * cs.pstride;
            if (k < M) { cs.kp0 = k; cs.P = (M - 1 - k) / cs.pstride + 1; }
        }
        cs.J = cs.A + cs.P;
        cs.wpos0 = full0 ? st.xi[c] : st.count[c];
        cs.newest0 = full0 ? (st.xi[c] + cap - 1) % cap : 0;
        cs.pre = (full0 && M > 0 && cs.kp0 > 0) ? 1 : 0;

        st.discards[c] += M - cs.A - cs.P;              // every SELECT loses one item
        if (c == g.N - 1) st.discards[c] += cs.P;       // evicted from the last cascade
        st.count[c] += cs.A;
        if (st.count[c] == cap) st.xi[c] = (int)(((int64_t)(full0 ? st.xi[c] : 0) + cs.P) % cap);

        if (cs.P > 0) { first += (int64_t)cs.kp0 * step; step *= cs.pstride; }
        M = cs.P;
    }
    st.t += Qc;
    st.n_seen += Q;
    st.sink_fill += plan.n_to_sink;
}

// Fixed tiles, xi the first row of one: rows of the oldest part in front of the extra cut (0: nothing to cut).
static int cut_of(int cap, int xi) { return std::min(32, (cap - xi) / 2); }

// Cache order is sinks, last cascade oldest..newest, ..., first cascade (Section 3.1
// "Positional Encoding": the index inside the cache).  Stored keys are rotated to their
// physical slot index, so within a run where (cache index - slot index) is constant the
// queries need one rotation: by (own index) - (that constant).  The segments are listed in
// physical order (the wrapped part of a ring before its oldest part): attention does not care
// in which order it meets the keys, but for the rounding of its sums, and a full cache then always reads front to back.  The
// wrapped part of a full ring is listed as [0, o) and [o, xi), o = xi mod 64, which fixes the
// place of every 64-row tile of the ring (see PackedLayout, also for the other cut).
void build_segments(const Geom& g, const HostState& st, bool with_chunk, int Q, SegList& out, bool fixed)
{
    out.n = 0;
    out.n_qvar = 0;
    const int n = st.n_cached(g);
    out.n_cached = n;
    auto add = [&](int start, int len, int delta, int chunk, int pad = 0) {
        if (len <= 0) return;
        const int rot0 = n - delta;
        int v = -1;
        for (int i = 0; i < out.n_qvar; ++i) if (out.qrot0[i] == rot0) v = i;
        if (v < 0) { v = out.n_qvar++; out.qrot0[v] = rot0; }
        out.pad[out.n] = pad;
        Seg& s = out.s[out.n++];
        s.start = start; s.len = len; s.qvar = v; s.chunk = chunk;
    };
    add(0, st.sink_fill, 0, 0);
    int rank = st.sink_fill;                         // cache index of the oldest item of the cascade
    for (int c = g.N - 1; c >= 0; --c) {
        const int cnt = st.count[c], cap = g.cap[c], xi = st.xi[c], base = g.base[c];
        if (cnt < cap) {
            add(base, cnt, rank - base, 0);
        } else {
            if (fixed) {
                const int o = xi % 64, cut = o ? 0 : cut_of(cap, xi), oldest = rank - (base + xi);
                add(base, xi, rank + (cap - xi) - base, 0);
                add(base + xi, cut, oldest, 0);
                add(base + xi + cut, cap - xi - cut, oldest, 0, o + cut);
                rank += cnt;
                continue;
            }
            const int o = with_chunk ? xi % 64 : 0, wrapped = rank + (cap - xi) - base;
            add(base, o, wrapped, 0);                                 // wrapped part: ring [0, xi), in two pieces (packed tiles only)
            add(base + o, xi - o, wrapped, 0);
            add(base + xi, cap - xi, rank - (base + xi), 0);          // oldest part: ring [xi, cap)
        }
        rank += cnt;
    }
    if (with_chunk) add(0, Q, n, 1);                 // chunk key i is rotated to i and sits at n + i
    int tiles = 0;
    for (int i = 0; i < kMaxSegments; ++i) {
        out.tile0[i] = i < out.n ? tiles : INT32_MAX;
        if (i < out.n) tiles += (out.s[i].len + out.pad[i] + 63) / 64;
    }
}

void plan_insert(const Geom& g, const UpdatePlan& plan, DecodeInsert& out)
{
    out = DecodeInsert();
    out.id0 = plan.id0;
    auto add = [&](int kind, int slot) { out.kinds |= (uint32_t)kind << (2 * out.n); out.slot[out.n] = slot; ++out.n; };
    if (plan.n_to_sink > 0) {
        add(kInsertAppend, plan.sink_fill0);
        return;
    }
    for (int c = 0; c < g.N && plan.c[c].M > 0; ++c) {
        const CascStep& cs = plan.c[c];
        if (cs.A > 0) add(kInsertAppend, cs.base + cs.wpos0);
        else if (cs.P > 0) add(kInsertPush, cs.base + cs.wpos0);
        else add(kInsertCompete, cs.base + cs.newest0);
    }
}

void plan_trees(const UpdatePlan& plan, int capacity, MoveTrees& out)
{
    out = MoveTrees();
    auto add = [&](int c, int lo, int count, int per) {
        if (count <= 0) return;
        out.c[out.n] = c; out.lo[out.n] = lo; out.count[out.n] = count; out.per[out.n] = per; out.first_wg[out.n] = out.wgs;
        out.wgs += (count + per - 1) / per;
        ++out.n;
    };
    long size = 0;                                   // at most this many slots hang on a slot of the cascade, itself included
    for (int c = 0; c < plan.N && plan.c[c].M > 0; ++c) {
        const CascStep& cs = plan.c[c];
        // offers to one slot: until the first push for the newest item and the last append, a stride for a push
        int offers = 1;
        if (cs.pre) offers = std::max(offers, cs.kp0);
        if (cs.A > 0) offers = std::max(offers, cs.kp0 - (cs.A - 1));
        if (cs.P > 0) offers = std::max(offers, cs.pstride);
        size = c == 0 ? 1 : 1 + std::min(offers, cs.M) * size;
        const bool last = c + 1 == plan.N || plan.c[c + 1].M == 0;
        const int roots = cs.pre + (last ? cs.J : cs.A);
        if (roots > 0 && size > capacity) { out = MoveTrees(); return; }
        add(c, -cs.pre, roots, (int)(capacity / size));
    }
    add(-1, 0, plan.n_to_sink, capacity);
}

// Splits of a decode step: as many as make the busiest compute unit finish first.  A CU holds one workgroup of
// the bf16 kernels (their rings fill the LDS); a workgroup costs about as much as two rounds of four tiles besides (first
// copies, queries, epilogue).  Where the shares differ by a tile, half a tile is charged.  Where even then there are hundreds
// of tiles for each of four waves, more rounds even out the CUs.  All of this was fitted to kernels of four waves, which the bf16
// ones no longer are.  With the present kernels, the rule's count / the best of up to 22, us a step in a stream of steps (in
// brackets the best count where the rule is off by more than 2 %):
// bf16, d = 128, 4 query heads: 8 KV heads: 4K slots 11.0 / 11.2, 8K 13.3 / 12.8 (24), 16K 16.8 / 16.9, 64K 51.5 / 49.2 (24); 16 heads
// of 8K 17.8 / 17.7; 64 of 16K 96.2 / 93.7 (3); 128 of 4K 52.2 / 52.0; 256 of 2K 55.9 / 56.4, of 8K 198 / 197, of 64K 1526 / 1523 (one
// split 1530); one head of 64K 21.4 / 16.7 (128).  One query head: 64 of 16K 88.0 / 87.9, 256 of 8K 189 / 183 (6).  Eight: 102.2 / 102.0,
// 217 / 212 (3).  d = 64: 8 heads of 16K 13.2 / 12.7 (28), 64 of 16K 57.2 / 54.5 (3), 128 of 4K 30.7 / 30.5, 512 of 4K 119 / 120.
// fp32 (four tiles at a time): d = 128: 8 heads of 4K 42.4 / 42.0, of 16K 33.2 / 33.5 (one query head), 64 of 4K 105 / 109, 256 of 2K
// 248 / 253; d = 64: 8 of 4K 27.7 / 27.7, 64 of 4K 76.3 / 52.2 (12), 256 of 2K 167 / 98 (3).
// For a given number of rounds the cost falls with every split, so only the most splits of each number of
// rounds are looked at: nine at most, 0.05 us of host time a step (all of up to 2048 split counts: 9.7).
int decode_split_count(int pairs, int most, int n_tiles)
{
    constexpr int kWaves = 4, kCus = 256;     // (four tiles at a time, as in fp32; the bf16 kernels take eight)
    if (n_tiles == 0) return 1;
    int best = 1;
    float best_cost = -1.f;
    int s = 0;
    for (long rounds = (pairs + kCus - 1) / kCus; s < most; ++rounds) {
        const int fit = (int)std::min((long)most, kCus * rounds / pairs);
        if (fit <= s) continue;
        s = fit;
        const long used = (pairs * (long)s + kCus - 1) / kCus, tiles = (n_tiles + s - 1) / s;
        const float share = (float)n_tiles / (float)(s * kWaves);
        const float cost = (float)used * (0.5f * ((float)((tiles + kWaves - 1) / kWaves) + share) + 2.f);
        if (best_cost < 0.f || cost < best_cost) { best = s; best_cost = cost; }
    }
    while (2 * best <= most && n_tiles / (2 * best * kWaves) >= 64) best *= 2;
    return best;
}

void packed_layout(const Geom& g, const HostState& st, PackedLayout& out, bool fixed)
{
    out.fixed = fixed;
    out.full = st.sink_fill == g.n_sink;
    int tiles = (g.n_sink + 63) / 64;
    for (int c = g.N - 1; c >= 0; --c) {             // physical order: the last cascade first
        if (st.count[c] != g.cap[c]) out.full = false;
        const int o = st.xi[c] % 64;
        out.off[c] = o;
        out.tile0[c] = tiles;
        tiles += fixed ? 1 + (g.cap[c] + 63) / 64 : (o > 0 ? 1 : 0) + (g.cap[c] - o + 63) / 64;
    }
    out.cache_tiles = tiles;
}

bool same_offsets(const Geom& g, const PackedLayout& a, const PackedLayout& b)
{
    for (int c = 0; c < g.N; ++c) if (a.off[c] != b.off[c]) return false;
    return true;
}

// Packing everything costs a read and a write of all cached rows (16K slots 31 us, 64K 100; us a call with and without
// fixed tiles, one context: 16 tokens against 64K slots 254 -> 169, 64 against 16K 103 -> 86).  The cut by offset
// has no tile more than it needs and keeps its tiles when a chunk moves every ring by whole tiles; any other
// chunk changes the offsets and starts with fixed tiles, which stay in use until something else
// (a decode step, an update that was not followed) makes the copies invalid.  The cut does not depend on whether the
// copies can be kept at all: contexts that share them (the layers of one workspace) follow the same rule and get the
// same sums, but pack everything for every chunk either way.
void plan_packing(const Geom& g, const HostState& st, int Q, const PackedCopies& pc, SegList& sl, PackedLayout& lay, TileRuns& runs)
{
    packed_layout(g, st, lay, false);
    bool partial = false;
    if (lay.full) {
        bool possible = pc.may_fix;      // (a last row that begins a tile cannot be cut)
        for (int c = 0; c < g.N; ++c) possible = possible && (st.xi[c] % 64 != 0 || cut_of(g.cap[c], st.xi[c]) > 0);
        if (pc.valid && !pc.lay.fixed && same_offsets(g, lay, pc.lay)) partial = true;
        else if (possible) {
            bool fixed = pc.valid && pc.lay.fixed;
            partial = fixed;
            if (!fixed) {
                HostState next = st;
                UpdatePlan pl;
                PackedLayout after;
                plan_update(g, next, Q, pl);
                packed_layout(g, next, after, false);
                fixed = !same_offsets(g, lay, after);
            }
            if (fixed) packed_layout(g, st, lay, true);
        }
    }
    build_segments(g, st, true, Q, sl, lay.fixed);
    const int chunk_tiles = (Q + 63) / 64;
    if (partial && pc.own && pc.reuse) {
        runs = pc.stale;
        if (add_tile_run(runs, lay.cache_tiles, chunk_tiles)) return;
    }
    int tiles = 0;
    for (int i = 0; i < sl.n; ++i) tiles += (sl.s[i].len + sl.pad[i] + 63) / 64;
    runs.n = 0;
    runs.total = 0;
    add_tile_run(runs, 0, tiles);
}

void packed_after_update(const Geom& g, const PackedLayout& lay, const HostState& before, const HostState& after, const UpdatePlan& pl, PackedCopies& pc)
{
    pc.valid = false;
    if (!lay.full) return;
    pc.lay = lay;
    pc.stale.n = 0;
    pc.stale.total = 0;
    pc.valid = true;
    if (!lay.fixed) {
        pc.valid = add_touched_tiles(g, lay, pl, pc.stale);
        return;
    }
    for (int c = 0; c < pl.N && pl.c[c].M > 0; ++c) {
        const CascStep& cs = pl.c[c];
        const int xi = before.xi[c], tiles = 1 + (cs.cap + 63) / 64;
        if (cs.J + cs.pre == 0) continue;
        // from the first row written to the tile the ring head now stands in, second listing included; a ring
        // that starts over, or whose newest item is its last row, is packed anew
        int first = 0, last = tiles - 1;
        if (!(xi + cs.J >= cs.cap || (cs.pre && xi == 0))) {
            first = (xi - cs.pre) / 64;
            last = std::min(last, after.xi[c] / 64 + 1);
        }
        pc.valid = pc.valid && add_tile_run(pc.stale, lay.tile0[c] + first, last - first + 1);
    }
}

static int tile_of_slot(const Geom& g, const PackedLayout& lay, int slot)
{
    if (slot < g.n_sink) return slot / 64;
    for (int c = 0; c < g.N; ++c) {
        const int r = slot - g.base[c];
        if (r < 0 || r >= g.cap[c]) continue;
        const int o = lay.off[c];
        return lay.tile0[c] + (r < o ? 0 : (o > 0 ? 1 : 0) + (r - o) / 64);
    }
    return -1;
}

int touched_slot_runs(const Geom& g, const UpdatePlan& pl, int* lo, int* hi)
{
    int n = 0;
    if (pl.n_to_sink > 0) { lo[n] = pl.sink_fill0; hi[n] = pl.sink_fill0 + pl.n_to_sink; ++n; }
    for (int c = 0; c < pl.N; ++c) {
        const CascStep& cs = pl.c[c];
        if (cs.M == 0) break;
        // ring positions wpos0 .. wpos0 + J - 1 are opened; before the first push the offers
        // compete with the item at newest0 = wpos0 - 1
        const int len = cs.J + cs.pre;
        if (len == 0) continue;
        if (len >= cs.cap) { lo[n] = cs.base; hi[n] = cs.base + cs.cap; ++n; continue; }
        const int start = cs.pre ? cs.newest0 : cs.wpos0;
        const int end = start + len;
        if (end <= cs.cap) { lo[n] = cs.base + start; hi[n] = cs.base + end; ++n; }
        else {
            lo[n] = cs.base + start; hi[n] = cs.base + cs.cap; ++n;
            lo[n] = cs.base; hi[n] = cs.base + end - cs.cap; ++n;
        }
    }
    return n;
}

bool add_tile_run(TileRuns& runs, int first, int count)
{
    if (count <= 0) return true;
    if (runs.n == kMaxTileRuns) return false;
    runs.first[runs.n] = first;
    runs.ahead[runs.n] = runs.total;
    runs.total += count;
    ++runs.n;
    return true;
}

bool add_touched_tiles(const Geom& g, const PackedLayout& layout, const UpdatePlan& pl, TileRuns& runs)
{
    int lo[kMaxTileRuns], hi[kMaxTileRuns];
    const int n = touched_slot_runs(g, pl, lo, hi);
    for (int i = 0; i < n; ++i) {                    // a run lies inside one ring: its tiles are consecutive
        const int t0 = tile_of_slot(g, layout, lo[i]), t1 = tile_of_slot(g, layout, hi[i] - 1);
        if (t0 < 0 || t1 < t0 || !add_tile_run(runs, t0, t1 - t0 + 1)) return false;
    }
    return true;
}

int slot_of_rank(const Geom& g, const HostState& st, int r)
{
    if (r < st.sink_fill) return r;
    r -= st.sink_fill;
    for (int c = g.N - 1; c >= 0; --c) {
        const int cnt = st.count[c];
        if (r < cnt) return g.base[c] + (cnt < g.cap[c] ? r : (st.xi[c] + r) % g.cap[c]);
        r -= cnt;
    }
    return -1;
}

}  // namespace ckv
