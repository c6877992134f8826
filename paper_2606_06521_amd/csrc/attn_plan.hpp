// Which kernel a call runs on and how it is cut into workgroups.  Host code
// without HIP, so that tests can ask for the choice.
#pragma once

#include <math.h>
#include <stddef.h>

#include <algorithm>

namespace attn {

constexpr int kNumXcd = 8;   // MI355X: 8 XCDs x 32 CUs, workgroup i runs on XCD i % 8

// query rows per tile of the fast kernel (one work unit of the 128-row schedule,
// half of one of the 256-row schedule's tile pairs)
constexpr int kFastRows = 256;
constexpr int kFastRowsPair = 128;

struct Shape {
    long long B, Hq, Hkv, N, Nk;   // N query rows, the last of Nk positions
    int d, block_kv;
    bool causal, qk8, count;       // qk8: E4M3 Q and K; count: with the P-underflow counts
};

// Queries against a longer KV cache whose split may use a workspace: short
// chunks, and long ones that start inside a block.
inline bool kv_may_split(const Shape& p)
{
    return p.Nk != p.N && (p.N < 128 || (p.Nk - p.N) % p.block_kv != 0);
}

// ---- the KV-cache kernel ----

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int kMaxRanges = 512;   // nsplit * tile height (range maxima staged by one workgroup)

// Two workgroups per tile that share its columns: where no shape makes them the
// shortest (d = 64 and small blocks leave each too little), they are not built.
constexpr bool kv_cols_built(int d, int block_kv, bool qk8, int waves)
{
    return d == 128 ? waves == 8 || !qk8 || block_kv == 128 : waves == 8 && !(qk8 && block_kv == 64);
}

struct KvPlan {
    int rows;              // tile height
    int cols;              // workgroups per tile that share its columns (unsplit tiles)
    int waves;             // per workgroup
    long long run;         // rows that share tiles: a group's, or one head's (causal heads of 128 rows or more)
    long long tiles;       // per (batch, KV head)
    long long units;
    long long C;           // workgroups per tile that share its keys
    long long slots;       // workgroups per XCD
    size_t off_part, bytes;   // workspace: where the partial sums start, and its size
    double time_us;        // expected
};

inline void plan_bytes(KvPlan& pl, int d)
{
    pl.off_part = pl.bytes = 0;
    if (pl.C > 1) {
        pl.off_part = align256((size_t)pl.units * pl.C * pl.rows * sizeof(float));
        pl.bytes = pl.off_part + align256((size_t)pl.units * pl.C * (pl.rows * (size_t)d + pl.rows) * sizeof(float));
    }
}

// The candidates -- 16- or 32-row tiles on workgroups of eight or four waves,
// unsplit, by two workgroups per tile that share its columns, or by C ranges of
// its keys -- by their time from what was measured of each part (us, bytes per
// us):
// - a launch of eight-wave workgroups costs 7, of four-wave ones 5, the three of
//   a split 15, and 4 more for every further generation of workgroups (their
//   start and merge); a CU holds one workgroup of eight waves or two of four;
// - every workgroup reads its tile's K (twice in a split: range maxima first)
//   and V, in rounds of a block per wave: 75 000 from the CU's L2 (tiles of one
//   head side by side: 64 queries of 4 x 32 heads against 8192 keys, 49 us).  A
//   round of 128-key blocks takes a full CU at least 4.8 on 32-row tiles (their
//   softmax; 2048 x 2048, 8 heads, E4M3: 31 us), 2.6 on 16-row ones, four waves
//   alone on their CU 4.0 and 3.0 (the same 64 queries: 69 us), and 2 whatever
//   the block (777 x 777, d = 64, blocks of 64: 17 us).  The long visits of a
//   split at d = 64 show less: 3.4 on 32-row tiles, 1.5 whatever the block (13 x 4/1
//   heads x 64 queries x 58454 E4M3 keys, blocks of 64: 144 us split, 186 unsplit),
//   and so do two workgroups of four waves with E4M3 scores (16/4 heads x 1995
//   queries x 3914 keys: 37 us, the fast kernel 63);
// - a (batch, KV head)'s keys come from HBM once: 40 000 per CU (decode of 16
//   requests x 8 KV heads x 8192 keys on 128 CUs: 4.7 TB/s), 33 000 with four
//   waves on it, 6 200 000 in all.  Keys that the Infinity Cache cannot keep from
//   call to call (96 MB and more) also cost the further reads of a range, by the
//   tiles of its head: 75 000 per CU and a fifth of the first one's share of the
//   total (5 x 8 heads x 32 queries x 95011 keys: 16-row tiles 300 us, 32-row
//   ones 250).  Two workgroups that share a tile's columns go through its K at
//   the same pace, so that each counts in full, 43 000 per CU (61 x 16384 keys on
//   122 CUs: 124 us; split in four 104), 49 000 where a head has several tiles (64 x
//   32 queries x 4096 keys: 33 us on 256 CUs, one workgroup per tile 36);
// - the counts take about a sixth more everywhere but on 32-row tiles with bf16
//   scores at d = 128, blocks of 128, whose kernel spills (4096 x 4096, 4 heads: 51
//   us, with counts 75, on 16-row tiles 76 and 81; the fast kernel 51 and 62; 2048 x
//   2048, 8 heads: 24 and 39): half more and 2 unsplit, 1.4 times split (the range
//   maxima take no counts).
// C = min(n_cu / units, blocks / 8, 512 / rows): every wave still has a block.
inline KvPlan kv_plan(const Shape& p, int n_cu, size_t ws_bytes)
{
    const int d = p.d, block_kv = p.block_kv;
    const long long rows = p.Hq / p.Hkv * p.N;
    // (fewer rows lie within 128 positions, as the rows of one block do)
    const long long run = p.causal && p.N >= 128 ? p.N : rows;
    const long long nb = (p.Nk + block_kv - 1) / block_kv;   // (no tile visits more blocks than this)
    const double k_row = p.qk8 ? d : 2 * d, v_row = d;
    const double head_keys = (double)p.B * p.Hkv * nb * block_kv;
    // one pass over `row` bytes per key on wgs workgroups of `blocks` blocks each
    const bool spills = p.count && !p.qk8 && d == 128 && block_kv == 128;
    const bool cached = head_keys * (k_row + v_row) <= 96e6;
    auto pass = [&](const KvPlan& pl, double wgs, double blocks, double row) {
        const double per_cu = 8 / pl.waves, gens = ceil(wgs / (n_cu * per_cu));
        const double here = std::min(ceil(wgs / n_cu), per_cu), active = std::min(wgs, (double)n_cu);
        const bool maxima = row == k_row, solo = here < per_cu;
        const double small = d == 64 && (pl.C > 1 || (pl.rows == 32 && pl.waves == 4 && p.qk8)) ? 0.7 : 1;
        const double full = maxima ? 0 : pl.rows == 32 ? 4.8 * small : 2.6, alone = pl.rows == 32 ? 4.0 : 3.0;
        const double round = std::max({here * pl.waves * block_kv * row / 75e3, full * here / per_cu * block_kv / 128,
                                       solo ? alone * block_kv / 128 : 0, small < 1 ? 1.5 : 2.0});
        const double once = head_keys * (maxima ? k_row : k_row + v_row), cu = solo ? 33e3 : 40e3;
        double mem = once / std::min(6.2e6, cu * active);
        if (!cached) {
            const double all = std::max(once, wgs * blocks * block_kv * row), again = all - once;
            const double pairs = (pl.tiles > 1 ? 49e3 : 43e3) / 40e3 * cu;
            mem = std::max((once + again / 5) / 6.2e6,
                           (pl.cols == 2 ? all / pairs : once / cu + again / 75e3) / active);
        }
        return std::max(gens * ceil(blocks / pl.waves) * round + 4 * (gens - 1), mem);
    };
    KvPlan best{};
    for (int tr = 16; tr <= (rows > 16 ? 32 : 16); tr *= 2) {
        KvPlan pl{};
        pl.rows = tr;
        pl.C = 1;
        pl.run = run;
        pl.tiles = rows / run * ((run + tr - 1) / tr);
        pl.units = p.B * p.Hkv * pl.tiles;
        auto take = [&](double t) {
            if (spills && tr == 32)
                t = pl.C > 1 ? 1.4 * t : 1.5 * t + 2;
            if (best.rows == 0 || t < best.time_us) {
                best = pl;
                best.time_us = t;
            }
        };
        for (pl.waves = 8; pl.waves >= 4; pl.waves /= 2) {
            const double launch = pl.waves == 8 ? 7 : 5;
            pl.cols = 1;
            take(launch + pass(pl, (double)pl.units, (double)nb, k_row + v_row));
            if (tr == 16 && 2 * pl.units <= n_cu && kv_cols_built(d, block_kv, p.qk8, pl.waves)) {
                pl.cols = 2;
                take(launch + pass(pl, 2.0 * pl.units, (double)nb, k_row + v_row / 2));
            }
        }
        pl.waves = 8;
        pl.cols = 1;
        pl.C = std::min({n_cu / pl.units, nb / pl.waves, (long long)(kMaxRanges / tr)});
        for (; pl.C > 1; --pl.C) {
            plan_bytes(pl, d);
            if (pl.bytes <= ws_bytes)
                break;
        }
        if (pl.C > 1) {
            const double wgs = (double)pl.units * pl.C, blocks = ceil((double)nb / pl.C);
            take(15 + pass(pl, wgs, blocks, k_row) + pass(pl, wgs, blocks, k_row + v_row));
        }
    }
    plan_bytes(best, d);
    // (the workgroups that share a tile's columns stay on one XCD)
    best.slots = (best.units * best.C + kNumXcd - 1) / kNumXcd * best.cols;
    return best;
}

// The least a caller's workspace has to hold: what a split of 32-row tiles
// per query head over min(n_cu / tiles, blocks / 8, 8) workgroups takes (a plan
// that could use more makes do with what it is given).
inline size_t kv_workspace_min(const Shape& p, int n_cu)
{
    const long long units = p.B * p.Hq * ((p.N + 31) / 32);
    const long long nb = (p.Nk + p.block_kv - 1) / p.block_kv;
    if (!kv_may_split(p) || units >= n_cu)
        return 0;
    const long long C = std::min({n_cu / units, nb / 8, 8LL});
    if (C <= 1)
        return 0;
    return align256((size_t)units * C * 8 * 32 * sizeof(float)) +
           align256((size_t)units * C * (32 * (size_t)p.d + 32) * sizeof(float));
}

// What a call can use.
inline size_t kv_workspace_bytes(const Shape& p, int n_cu)
{
    if (!kv_may_split(p))
        return 0;
    size_t bytes = kv_workspace_min(p, n_cu);
    for (const bool count : {false, true}) {   // (one size for a shape's calls with and without counts)
        Shape s = p;
        s.count = count;
        bytes = std::max(bytes, kv_plan(s, n_cu, ~(size_t)0).bytes);
    }
    return bytes;
}

// ---- the fast kernel ----

// Critical path of the fast kernel's persistent grid on one schedule, in
// ping-pong phases: the largest sum of unit costs any workgroup takes, with
// the kernel's assignment (XCD x owns units [units x / 8, units (x + 1) / 8),
// its workgroups take every per-th of them).  A tile of the 256-row schedule
// costs two phases per visited block (plus one block's worth for the last
// P.V); one of the 128-row schedule one phase per block (plus two), times
// kPairPhase, the measured length of its phases against the 256-row
// schedule's (every phase of the 128-row schedule carries a K/V copy burst).
constexpr double kPairPhase = 1.15;

inline double fast_critical_path(const Shape& p, bool pair, int n_cu)
{
    const int rows = pair ? kFastRowsPair : kFastRows;
    const long long T = (p.N + rows - 1) / rows;
    const long long per_head = pair ? T : (T + 1) / 2;
    const long long units = p.B * p.Hq * per_head;
    auto tile_cost = [&](long long t) {
        const long long last = std::min((t + 1) * rows, p.N) - 1;
        const long long nb = p.causal ? (last + p.Nk - p.N) / p.block_kv + 1 : (p.Nk + p.block_kv - 1) / p.block_kv;
        return pair ? (double)(nb + 2) * kPairPhase : 2.0 * (double)(nb + 1);
    };
    auto unit_cost = [&](long long u) {
        const long long pr = u % per_head;
        if (pair)
            return tile_cost(pr);
        const long long a = T - 1 - pr;
        return a == pr ? tile_cost(pr) : tile_cost(a) + tile_cost(pr);
    };
    const long long per_xcd_max = n_cu >= kNumXcd ? n_cu / kNumXcd : 1;
    const long long per = std::min(units / kNumXcd + 1, per_xcd_max);
    double worst = 0.0;
    for (int x = 0; x < kNumXcd; ++x) {
        const long long b = units * x / kNumXcd, e = units * (x + 1) / kNumXcd;
        for (long long slot = 0; slot < per; ++slot) {
            double sum = 0.0;
            for (long long u = b + slot; u < e; u += per)
                sum += unit_cost(u);
            worst = std::max(worst, sum);
        }
    }
    return worst;
}

struct Route {
    bool kv;      // the KV-cache kernel, by plan
    bool pair;    // otherwise the fast kernel: its 128-row schedule
    int row_lo;   // ... and the empty rows before a causal chunk that starts inside a block
    KvPlan plan;
};

// Kernel and schedule of a fast-mode call.  Fewer than 128 queries against a
// cache: the KV-cache kernel.  Otherwise 256-row tiles in causal-balanced pairs on
// the fast kernel, unless the caller asked otherwise (tile 128 or 256; diag: the
// per-block diagnostic, which only the fast kernel takes) or their units leave CUs
// idle: then the shortest, by their models, of those, the 128-row schedule (one
// tile per unit, two waves per 32-row group) and the KV-cache kernel.  A path of
// the fast kernel costs 6.5 us and, per phase of a block of 128 keys at d = 128,
// 1.3 (4096 x 4096 keys, 2 heads: 51 us for 39 phases, the KV-cache kernel 30;
// 512 x 512, 8 heads, causal: 17 for 7, and 10).
inline Route fast_route(const Shape& p, int tile, bool diag, int n_cu, size_t ws_bytes)
{
    Route r{};
    const size_t kv_ws = kv_may_split(p) ? ws_bytes : 0;
    if (p.Nk != p.N && p.N < 128) {
        r.kv = true;
        r.plan = kv_plan(p, n_cu, kv_ws);
        return r;
    }
    // The fast kernel's causal rows start at a block boundary: a chunk that starts
    // inside a block is preceded by row_lo empty rows (fewer than a block).
    Shape f = p;
    r.row_lo = p.causal ? (int)((p.Nk - p.N) % p.block_kv) : 0;
    f.N += r.row_lo;
    r.pair = tile == kFastRowsPair;
    const long long tiles = (f.N + kFastRows - 1) / kFastRows;
    if (tile == 0 && p.B * p.Hq * ((tiles + 1) / 2) < n_cu) {
        const double t256 = fast_critical_path(f, false, n_cu), t128 = fast_critical_path(f, true, n_cu);
        r.pair = t128 < t256;
        if (!diag) {
            const double phase = (0.25 + 1.05 * p.block_kv / 128 * (p.d == 64 ? 0.6 : p.qk8 ? 0.8 : 1.0)) *
                                 (p.count ? 1.17 : 1.0);
            r.plan = kv_plan(p, n_cu, kv_ws);
            r.kv = r.plan.time_us < 6.5 + phase * std::min(t128, t256);
        }
    }
    return r;
}

}  // namespace attn
