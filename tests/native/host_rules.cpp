// Test infrastructure: rules of the library's host side (structure.cpp) driven directly, without a device.
//   packing SEED   which tiles of the packed K / V copies a chunk packs again: a replay of a random geometry that
//                  packs token numbers in the place of rows.  Exit code 0 = every row is where it is read.
//   trees SEED     the update of a chunk in trees: workgroup after workgroup in a drawn order, each reading its slots' new
//                  rows from the cache as it then is and writing them, against Alg. 2 token by token.
//   large D CHUNK SIZE:PERIOD ...   how many updates of full chunks on a full cache are direct, with trees larger than any workgroup takes.
//   shares         where the shares of workgroups that divide the tiles of a row block begin, against 64-bit arithmetic.
//   splits         the split count of a decode step against the same costs looked at for every count, and its time.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <string>
#include <vector>

#include "../../paper_2406_17808_amd/csrc/plan_core.h"
#include "../../paper_2406_17808_amd/csrc/structure.h"

using namespace ckv;

static uint64_t rng_state;
static uint32_t rnd(uint32_t n)   // splitmix64, value in [0, n)
{
    uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (uint32_t)(z % n);
}

// ------------------------------------------------------------------ packed tiles

// Alg. 2 token by token on physical slots; whether an offer beats the newest item is drawn.
struct Rows {
    std::vector<int> id;
    std::vector<int> count, head;
    int sinks = 0;
    long t = 0, seen = 0;
    void insert(const Geom& g, const cascade_config& cfg)
    {
        int x = (int)seen++;
        if (sinks < g.n_sink) { id[sinks++] = x; return; }
        const long now = t++;
        for (int c = 0; c < g.N; ++c) {
            const int base = g.base[c], cap = g.cap[c];
            if (count[c] < cap) { id[base + count[c]++] = x; return; }
            const int period = cfg.accept_period[0] ? cfg.accept_period[c] : 1 << c;
            if (now % period) {
                if (rnd(2)) id[base + (head[c] + cap - 1) % cap] = x;
                return;
            }
            std::swap(x, id[base + head[c]]);
            head[c] = (head[c] + 1) % cap;
        }
    }
};

// Packs what plan_packing names and looks whether every cached row is then where the attention kernel reads it.
static const char* pack(const Geom& g, const HostState& st, int Q, const PackedCopies& pc, const std::vector<int>& id,
                        std::vector<std::vector<int>>& packed, PackedLayout& lay, int max_tiles, long* tiles_packed)
{
    SegList sl;
    TileRuns runs;
    plan_packing(g, st, Q, pc, sl, lay, runs);
    int n = 0, rows = 0, total = 0, last_start = -1;
    const char* wrong = nullptr;
    for (int i = 0; i < sl.n; ++i) {
        const Seg& sg = sl.s[i];
        if (!sg.chunk) rows += sg.len;
        // one order of the sums whatever the rings hold: another one moves the scores by their rounding, and with it
        // selections between tokens of almost equal score
        if (!sg.chunk && sg.start <= last_start) wrong = "the cached rows are not listed in the order of their slots";
        last_start = sg.start;
        if (sl.pad[i] < 0 || sl.pad[i] > 63 || sl.pad[i] > sg.start) wrong = "padding reaches outside the ring";
        for (int t0 = -sl.pad[i]; t0 < sg.len; t0 += 64, ++n) {
            if ((int)packed.size() <= n) packed.resize(n + 1, std::vector<int>(64, -2));
            bool now = false;
            for (int r = 0; r < runs.n; ++r) {
                const int end = (r + 1 < runs.n ? runs.ahead[r + 1] : runs.total) - runs.ahead[r];
                now = now || (n >= runs.first[r] && n < runs.first[r] + end);
            }
            total += now;
            if (sg.chunk && !now) wrong = "a tile of the chunk is not packed";
            for (int x = 0; x < 64 && !sg.chunk; ++x) {
                const bool in = t0 + x >= 0 && t0 + x < sg.len;
                if (now) packed[n][x] = in ? id[sg.start + t0 + x] : -2;
                if (in && packed[n][x] != id[sg.start + t0 + x]) wrong = "a packed tile does not hold the rows of its segment";
            }
        }
    }
    for (int r = 0; r < runs.n; ++r)
        if (runs.first[r] < 0 || runs.first[r] + (r + 1 < runs.n ? runs.ahead[r + 1] : runs.total) - runs.ahead[r] > n) wrong = "a run names tiles that do not exist";
    if (total > runs.total) wrong = "the runs hold fewer tiles than they name";
    if (rows != st.n_cached(g)) wrong = "the segments do not hold all cached rows";
    if (lay.full && n != lay.cache_tiles + (Q + 63) / 64) wrong = "the segments do not have the tiles of the layout";
    if (n > max_tiles) wrong = "more tiles than the workspace holds";
    *tiles_packed += runs.total;
    return wrong;
}

// kind 0: a context of its own; 1: copies shared between layers; 2: single-pass scores; 3: decode steps in between
static int packing_case(int seed, int kind, long* tiles_packed)
{
    rng_state = 0x1234567ull * (uint64_t)(seed + 1);
    static const int ring[] = {1, 2, 33, 64, 65, 97, 128, 192, 250, 320}, chunk[] = {1, 7, 16, 64, 100, 256}, sinks[] = {0, 3, 64};
    cascade_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.batch = 1; cfg.n_q_heads = 1; cfg.n_kv_heads = 1; cfg.head_dim = 64; cfg.dtype = CASCADE_BF16;
    cfg.n_sink = sinks[rnd(3)];
    cfg.n_cascades = 1 + (int)rnd(4);
    cfg.max_chunk = chunk[rnd(6)];
    cfg.ema_beta = 0.9f; cfg.rope_base = 10000.f;
    const bool periods = rnd(4) == 0;
    int largest = 0;
    for (int c = 0; c < cfg.n_cascades; ++c) {
        cfg.cascade_sizes[c] = ring[rnd(10)];
        cfg.accept_period[c] = periods ? (c == 0 ? 1 : 1 + (int)rnd(5)) : 0;
        largest = cfg.cascade_sizes[c] > largest ? cfg.cascade_sizes[c] : largest;
    }
    std::string why;
    if (check_config(&cfg, why) != CASCADE_OK) { fprintf(stderr, "seed %d: %s\n", seed, why.c_str()); return 1; }
    Geom g;
    make_geom(&cfg, g);
    Rows rows;
    rows.id.assign(g.slots, -1);
    rows.count.assign(g.N, 0);
    rows.head.assign(g.N, 0);
    HostState st;
    PackedCopies pc;
    pc.own = kind != 1;
    pc.may_fix = kind != 2;
    std::vector<std::vector<int>> packed;
    const int max_tiles = (g.slots + cfg.max_chunk) / 64 + kMaxSegments;
    int left = (largest << g.N) + 700;
    if (left > 6000) left = 6000;
    for (int step = 0; left > 0; ++step) {
        const int Q = rnd(10) < 7 ? cfg.max_chunk : 1 + (int)rnd(cfg.max_chunk);
        left -= Q;
        UpdatePlan pl;
        if (kind == 3 && rnd(3) == 0)
            for (int i = 1 + (int)rnd(3); i > 0; --i) {      // what a decode step does to the copies and the cache
                pc.valid = false;
                rows.insert(g, cfg);
                plan_update(g, st, 1, pl);
            }
        if (!pc.own) for (auto& tile : packed) tile.assign(64, -3);   // another layer has packed its own
        PackedLayout lay;
        const HostState before = st;
        const char* wrong = pack(g, st, Q, pc, rows.id, packed, lay, max_tiles, tiles_packed);
        if (wrong) { fprintf(stderr, "seed %d kind %d step %d: %s\n", seed, kind, step, wrong); return 1; }
        for (int i = 0; i < Q; ++i) rows.insert(g, cfg);
        plan_update(g, st, Q, pl);
        packed_after_update(g, lay, before, st, pl, pc);
        for (int c = 0; c < g.N; ++c)
            if (st.count[c] != rows.count[c] || (st.count[c] == g.cap[c] && st.xi[c] != rows.head[c])) { fprintf(stderr, "seed %d step %d: ring %d differs\n", seed, step, c); return 1; }
    }
    return 0;
}

// ------------------------------------------------------------------ updates in trees

struct Item { int id; float mu; };

static int trees_case(int seed, long* updates, long* refused)
{
    rng_state = 0x7654321ull * (uint64_t)(seed + 1);
    static const int ring[] = {1, 2, 7, 16, 33, 64, 100}, chunk[] = {1, 3, 16, 33, 64, 100}, sinks[] = {0, 3, 64}, room[] = {8, 16, 32, 64, 128, 256};
    cascade_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.batch = 1; cfg.n_q_heads = 1; cfg.n_kv_heads = 1; cfg.head_dim = 64; cfg.dtype = CASCADE_BF16;
    cfg.n_sink = sinks[rnd(3)];
    cfg.n_cascades = 1 + (int)rnd(8);
    cfg.max_chunk = chunk[rnd(6)];
    cfg.ema_beta = 0.9f; cfg.rope_base = 10000.f;
    cfg.token_selection = rnd(8) != 0;
    const bool periods = rnd(3) == 0, equal = rnd(2) == 0;
    for (int c = 0; c < cfg.n_cascades; ++c) {
        cfg.cascade_sizes[c] = equal ? 100 : ring[rnd(7)];
        cfg.accept_period[c] = periods ? (c == 0 ? 1 : 1 + (int)rnd(5)) : 0;
    }
    std::string why;
    if (check_config(&cfg, why) != CASCADE_OK) { fprintf(stderr, "seed %d: %s\n", seed, why.c_str()); return 1; }
    Geom g;
    make_geom(&cfg, g);
    std::vector<Item> cache(g.slots, Item{-1, 0.f});
    HostState st;
    for (int step = 0; step < 60; ++step) {
        const int Q = rnd(10) < 7 ? cfg.max_chunk : 1 + (int)rnd(cfg.max_chunk);
        std::vector<Item> fresh(Q);
        for (int i = 0; i < Q; ++i) fresh[i] = Item{(int)st.n_seen + i, (float)rnd(6)};     // ties
        // the chunk's scores replace those of the cached rows in a real call; here they stay
        std::vector<Item> want = cache;
        HostState one = st;
        for (int i = 0; i < Q; ++i) {
            Item x = fresh[i];
            UpdatePlan pl;
            DecodeInsert ins;
            plan_update(g, one, 1, pl);
            plan_insert(g, pl, ins);
            for (int e = 0; e < ins.n; ++e) {
                Item& there = want[ins.slot[e]];
                if (insert_kind(ins, e) != kInsertCompete) std::swap(x, there);
                else if (g.token_selection && x.mu > there.mu) there = x;
            }
        }
        UpdatePlan pl;
        plan_update(g, st, Q, pl);
        MoveTrees mt;
        const int capacity = room[rnd(6)];
        mt.wgs = 0;
        if (plan_is_direct(pl)) plan_trees(pl, capacity, mt);
        if (mt.wgs == 0) { cache = want; ++*refused; continue; }
        ++*updates;
        std::vector<float> mu(g.slots), muc(Q);
        for (int i = 0; i < g.slots; ++i) mu[i] = cache[i].mu;
        for (int i = 0; i < Q; ++i) muc[i] = fresh[i].mu;
        std::vector<int> order(mt.wgs);
        for (int i = 0; i < mt.wgs; ++i) order[i] = i;
        for (int i = mt.wgs - 1; i > 0; --i) std::swap(order[i], order[rnd(i + 1)]);
        for (int wg : order) {
            int cls = 0;
            while (cls + 1 < mt.n && wg >= mt.first_wg[cls + 1]) ++cls;
            const int r0 = (wg - mt.first_wg[cls]) * mt.per[cls], r1 = std::min(mt.count[cls], r0 + mt.per[cls]);
            std::vector<int> dst, ref;
            if (mt.c[cls] < 0)
                for (int x = r0; x < r1; ++x) { dst.push_back(pl.sink_fill0 + x); ref.push_back(g.slots + x); }
            else {
                int j0 = mt.lo[cls] + r0, j1 = mt.lo[cls] + r1;
                for (int c = mt.c[cls];; --c) {
                    for (int j = j0; j < j1; ++j) {
                        int sw;
                        // the scores as they are in the cache by now
                        for (int i = 0; i < g.slots; ++i) mu[i] = cache[i].mu;
                        ref.push_back(segment_winner(pl.c[c], c, j, g.slots, pl.n_to_sink, g.token_selection, nullptr, mu.data(), muc.data(), &sw, &pl));
                        dst.push_back(j < 0 ? pl.c[c].base + pl.c[c].newest0 : pl.c[c].base + (pl.c[c].wpos0 + j) % pl.c[c].cap);
                    }
                    if (c == 0) break;
                    child_segments(pl, c, &j0, &j1);
                }
            }
            if ((int)dst.size() > capacity) { fprintf(stderr, "seed %d step %d: %d slots for a workgroup of %d\n", seed, step, (int)dst.size(), capacity); return 1; }
            std::vector<Item> rows;
            for (int x : ref) rows.push_back(x < g.slots ? cache[x] : fresh[x - g.slots]);
            for (size_t i = 0; i < dst.size(); ++i) cache[dst[i]] = rows[i];
        }
        for (int i = 0; i < g.slots; ++i)
            if (cache[i].id != want[i].id || cache[i].mu != want[i].mu) { fprintf(stderr, "seed %d step %d: slot %d holds %d, not %d\n", seed, step, i, cache[i].id, want[i].id); return 1; }
    }
    return 0;
}

// Exit code 0: every one of 40 updates is direct and its trees are too large for 1024 threads, d / 16 for two slots.
static int large_trees(int argc, char** argv)
{
    cascade_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.batch = 1; cfg.n_q_heads = 1; cfg.n_kv_heads = 1; cfg.head_dim = atoi(argv[2]); cfg.dtype = CASCADE_F32;
    cfg.n_sink = 3; cfg.max_chunk = atoi(argv[3]); cfg.ema_beta = 0.9f; cfg.rope_base = 10000.f; cfg.token_selection = 1;
    for (int i = 4; i < argc; ++i, ++cfg.n_cascades)
        if (sscanf(argv[i], "%d:%d", &cfg.cascade_sizes[cfg.n_cascades], &cfg.accept_period[cfg.n_cascades]) != 2) return 2;
    std::string why;
    if (check_config(&cfg, why) != CASCADE_OK) { fprintf(stderr, "%s\n", why.c_str()); return 1; }
    Geom g;
    make_geom(&cfg, g);
    HostState st;
    UpdatePlan pl;
    while (st.n_cached(g) < g.slots) plan_update(g, st, cfg.max_chunk, pl);
    int large = 0;
    for (int i = 0; i < 40; ++i) {
        plan_update(g, st, cfg.max_chunk, pl);
        MoveTrees mt;
        plan_trees(pl, 1024 / (g.d / 16) * 2, mt);
        large += plan_is_direct(pl) && mt.wgs == 0;
    }
    printf("%d of 40 updates\n", large);
    return large == 40 ? 0 : 1;
}

// ------------------------------------------------------------------ shares of a row block's tiles

static int wrong_shares()
{
    const int most = (1 << 28) / 16 + 4096;          // 16-key tiles of the largest cache check_config accepts, and a chunk
    int bad = 0;
    for (int n = 1; n <= 256; ++n)
        for (int x : {1, 2, n - 1, n, n + 1, 2 * n + 1, 1000, (1 << 22) + 1, (1 << 23) - 1, 1 << 23, (1 << 23) + 77, 1 << 24, most - 1, most}) {
            if (x < 1) continue;
            for (int z = 0; z <= n; ++z) bad += share_begin(x, z, n) != (int)((int64_t)x * z / n);
        }
    return bad;
}

// ------------------------------------------------------------------ splits of a decode step

static int best_of_all_splits(int pairs, int most, int n_tiles)
{
    int best = 1;
    float best_cost = -1.f;
    for (int s = 1; s <= most; ++s) {
        const long rounds = (pairs * (long)s + 255) / 256, tiles = (n_tiles + s - 1) / s;
        const float cost = (float)rounds * (0.5f * ((float)((tiles + 3) / 4) + (float)n_tiles / (float)(s * 4)) + 2.f);
        if (best_cost < 0.f || cost < best_cost) { best = s; best_cost = cost; }
    }
    while (2 * best <= most && n_tiles / (8 * best) >= 64) best *= 2;
    return best;
}

static int splits_case()
{
    long n = 0, wrong = 0;
    for (int pairs = 1; pairs <= 2600; pairs = pairs < 300 ? pairs + 1 : pairs + 37)
        for (int slots = 1; slots < 1 << 21; slots = slots < 2000 ? slots + 331 : slots * 5 / 3 + 7) {
            int most = (2048 + pairs - 1) / pairs;         // the counts a workspace is laid out for
            if (most > (slots + 127) / 128) most = (slots + 127) / 128;
            for (int i = 0; i < 12; ++i, ++n) {
                const int tiles = i < 3 ? i : (int)((long)(slots / 32 + 9) * i / 11), got = decode_split_count(pairs, most, tiles);
                if (got != best_of_all_splits(pairs, most, tiles) && ++wrong <= 5)
                    fprintf(stderr, "%d pairs, %d splits at most, %d tiles: %d\n", pairs, most, tiles, got);
            }
        }
    double best = 1e9;
    for (int r = 0; r < 9; ++r) {
        long sum = 0;
        const auto t = std::chrono::steady_clock::now();
        for (int i = 0; i < 200; ++i) sum += decode_split_count(1, 2048, 8192 + i);
        const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() * 1e6 / 200;
        if (sum && us < best) best = us;
    }
    printf("%ld of %ld counts wrong, %.3f us a call\n", wrong, n, best);
    return wrong || best > 2.0 ? 1 : 0;       // a call of the whole step takes about ten
}

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "splits")) return splits_case();
    if (argc == 3 && !strcmp(argv[1], "packing")) {
        int bad = 0;
        long tiles[4] = {0, 0, 0, 0};
        for (int kind = 0; kind < 4; ++kind) bad += packing_case(atoi(argv[2]), kind, &tiles[kind]);
        printf("tiles packed: own %ld shared %ld single-pass %ld with decode steps %ld\n", tiles[0], tiles[1], tiles[2], tiles[3]);
        return bad ? 1 : 0;
    }
    if (argc == 3 && !strcmp(argv[1], "trees")) {
        long updates = 0, refused = 0;
        int bad = 0;
        for (int i = 0; i < 40; ++i) bad += trees_case(40 * atoi(argv[2]) + i, &updates, &refused);
        printf("%ld updates in trees, %ld not\n", updates, refused);
        return bad || updates < refused / 4 ? 1 : 0;
    }
    if (argc >= 5 && argc <= 4 + CASCADE_MAX_CASCADES && !strcmp(argv[1], "large")) return large_trees(argc, argv);
    if (argc == 2 && !strcmp(argv[1], "shares")) {
        const int bad = wrong_shares();
        printf("%d shares begin elsewhere\n", bad);
        return bad ? 1 : 0;
    }
    fprintf(stderr, "usage: host_rules packing SEED | trees SEED | large D CHUNK SIZE:PERIOD .. | shares | splits\n");
    return 2;
}
