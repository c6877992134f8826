// Launch plan of the KV-cache kernel (attn_prefill_kernel.hpp): tile height,
// split over workgroups, workspace, and the merge of a split tile.
#include "attn_common.hpp"
#include "attn_launch.hpp"

#include <math.h>

#include <algorithm>

namespace attn {

// Merge of a split tile: one workgroup of 256 threads per row; thread (piece,
// part) takes one 16-byte piece of the row from every PARTS-th of the nsplit
// partial sums, all requested at once, and the PARTS sums are added through LDS
// (a fixed order).  lse comes from the row's final maximum (the largest of its
// range maxima).  What bounds it is latency -- one round of loads, one of LDS:
// 32 partial sums of 32 rows 6.2 us with one thread per piece (four rounds of
// eight loads), 3.6 so.
template <int D, int TR>
__global__ void __launch_bounds__(256) prefill_merge(Params p)
{
    constexpr int PART = TR * D + TR;
    constexpr int PIECES = D / 4;               // 16-byte pieces per row
    constexpr int PARTS = 256 / PIECES;
    constexpr int CMAX = 512 / TR;              // largest nsplit
    constexpr int PER = (CMAX + PARTS - 1) / PARTS;
    __shared__ f32x4 osh[PARTS][PIECES];
    __shared__ float lsh[PARTS], msh[PARTS];
    const int C = p.nsplit;
    const int unit = blockIdx.x / TR, rr = blockIdx.x % TR;
    if (unit >= p.total_wg / C)
        return;
    const int bk = unit / p.n_tiles;
    const int tile = p.causal ? p.n_tiles - 1 - (unit - bk * p.n_tiles) : unit - bk * p.n_tiles;   // as kv_kernel
    const int run = tile / p.run_tiles;
    const int row = run * p.run + TR * (tile - run * p.run_tiles) + rr;
    if (row >= (run + 1) * p.run)
        return;
    const int piece = threadIdx.x % PIECES, part = threadIdx.x / PIECES;
    const float* base = p.ws_part + (size_t)unit * C * PART;
    const float* mx = p.ws_max + (size_t)unit * C * TR + rr;
    f32x4 x[PER];
    float lp[PER], mp[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = part + PARTS * i;
        const bool on = c < C;
        const float* b = base + (size_t)(on ? c : 0) * PART;
        x[i] = on ? *reinterpret_cast<const f32x4*>(b + rr * D + 4 * piece) : f32x4{};
        lp[i] = on ? b[TR * D + rr] : 0.f;
        mp[i] = on ? mx[c * TR] : -INFINITY;
    }
    f32x4 acc = x[0];
    float l = lp[0], m = mp[0];
#pragma unroll
    for (int i = 1; i < PER; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] += x[i][e];
        l += lp[i];
        m = fmax_f(m, mp[i]);
    }
    osh[part][piece] = acc;
    if (piece == 0) {
        lsh[part] = l;
        msh[part] = m;
    }
    __syncthreads();
    if (part != 0)
        return;
#pragma unroll
    for (int v = 1; v < PARTS; ++v) {
        const f32x4 t = osh[v][piece];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] += t[e];
        l += lsh[v];
        m = fmax_f(m, msh[v]);
    }
    // (l and m of part 0 are the same in all its pieces)
    const size_t flat = (size_t)bk * (p.Hq / p.Hkv * p.N) + row;
    if (p.out) {
        const float inv = p.v_descale / (p.S * l);
        f32x4 v4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v4[i] = acc[i] * inv;
        *reinterpret_cast<f32x4*>(p.out + flat * D + 4 * piece) = v4;
    }
    if (p.lse && piece == 0)
        p.lse[flat] = (m * p.c + __builtin_log2f(l)) * 0.6931471805599453f;
}

namespace {

// Clears the counts a split launch adds to.
__global__ void prefill_zero(uint32_t* a, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0u;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int kMaxRanges = 512;   // nsplit * tile height (range maxima staged by one workgroup)

struct Plan {
    int rows;              // tile height
    int cols;              // workgroups per tile that share its columns (unsplit tiles)
    int waves;             // per workgroup
    long long run;         // rows that share tiles: a group's, or one head's (causal heads of 128 rows or more)
    long long tiles;       // per (batch, KV head)
    long long units;
    long long C;           // workgroups per tile that share its keys
    size_t off_part, bytes;
};

void plan_bytes(Plan& pl, int d)
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
//   the block (777 x 777, d = 64, blocks of 64: 17 us);
// - a (batch, KV head)'s keys come from HBM once: 40 000 per CU (decode of 16
//   requests x 8 KV heads x 8192 keys on 128 CUs: 4.7 TB/s), 33 000 with four
//   waves on it, 6 200 000 in all.
// C = min(n_cu / units, blocks / 8, 512 / rows): every wave still has a block.
Plan make_plan(const Params& p, int d, int block_kv, bool causal, bool qk8, int n_cu, size_t ws_bytes,
               double* time = nullptr)
{
    const long long rows = (long long)p.Hq / p.Hkv * p.N;
    // (fewer rows lie within 128 positions, as the rows of one block do)
    const long long run = causal && p.N >= 128 ? p.N : rows;
    // (no tile visits more blocks than this)
    const long long nb = causal ? ((long long)p.N - 1 + p.qoff) / block_kv + 1
                                : ((long long)p.Nk + block_kv - 1) / block_kv;
    const double k_row = qk8 ? d : 2 * d, v_row = d;
    const double head_keys = (double)p.B * p.Hkv * nb * block_kv;
    // one pass over `row` bytes per key on wgs workgroups of `blocks` blocks each
    auto pass = [&](const Plan& pl, double wgs, double blocks, double row) {
        const double per_cu = 8 / pl.waves, gens = ceil(wgs / (n_cu * per_cu));
        const double here = std::min(ceil(wgs / n_cu), per_cu), active = std::min(wgs, (double)n_cu);
        const bool maxima = row == k_row, solo = here < per_cu;
        const double full = maxima ? 0 : pl.rows == 32 ? 4.8 : 2.6, alone = pl.rows == 32 ? 4.0 : 3.0;
        const double round = std::max({here * pl.waves * block_kv * row / 75e3, full * here / per_cu * block_kv / 128,
                                       solo ? alone * block_kv / 128 : 0, 2.0});
        return std::max(gens * ceil(blocks / pl.waves) * round + 4 * (gens - 1),
                        head_keys * (maxima ? k_row : k_row + v_row) / std::min(6.2e6, (solo ? 33e3 : 40e3) * active));
    };
    Plan best{};
    double t_best = 0;
    for (int tr = 16; tr <= (rows > 16 ? 32 : 16); tr *= 2) {
        Plan pl{};
        pl.rows = tr;
        pl.C = 1;
        pl.run = run;
        pl.tiles = rows / run * ((run + tr - 1) / tr);
        pl.units = (long long)p.B * p.Hkv * pl.tiles;
        auto take = [&](double t) {
            if (best.rows == 0 || t < t_best) {
                best = pl;
                t_best = t;
            }
        };
        for (pl.waves = 8; pl.waves >= 4; pl.waves /= 2) {
            const double launch = pl.waves == 8 ? 7 : 5;
            pl.cols = 1;
            take(launch + pass(pl, (double)pl.units, (double)nb, k_row + v_row));
            if (tr == 16 && 2 * pl.units <= n_cu) {
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
    if (time)
        *time = t_best;
    return best;
}

hipError_t launch_phase(const Params& p, const Plan& pl, int d, int block_kv, bool count, int scale, bool qk8,
                        int phase, hipStream_t s)
{
    auto go = [&](auto fn) { return fn(p, d, block_kv, count, scale, phase, pl.cols, pl.waves, s); };
    if (pl.rows == 16)
        return qk8 ? go(launch_kv_t<true, 16>) : go(launch_kv_t<false, 16>);
    return qk8 ? go(launch_kv_t<true, 32>) : go(launch_kv_t<false, 32>);
}

}  // namespace

double prefill_time_us(const Params& p, int d, int block_kv, bool causal, bool qk8, int n_cu, size_t ws_bytes)
{
    double t = 0;
    make_plan(p, d, block_kv, causal, qk8, n_cu, ws_bytes, &t);
    return t;
}

// The least a caller's workspace has to hold: what a split of 32-row tiles
// per query head over min(n_cu / tiles, blocks / 8, 8) workgroups takes (a plan
// that could use more makes do with what it is given).
size_t prefill_workspace_min(const Params& p, int d, int block_kv, bool causal, int n_cu)
{
    const long long units = (long long)p.B * p.Hq * ((p.N + 31) / 32);
    const long long nb = causal ? ((long long)p.N - 1 + p.qoff) / block_kv + 1
                                : ((long long)p.Nk + block_kv - 1) / block_kv;
    if (units >= n_cu)
        return 0;
    const long long C = std::min({n_cu / units, nb / 8, 8LL});
    if (C <= 1)
        return 0;
    return align256((size_t)units * C * 8 * 32 * sizeof(float)) +
           align256((size_t)units * C * (32 * (size_t)d + 32) * sizeof(float));
}

size_t prefill_workspace_bytes(const Params& p, int d, int block_kv, bool causal, bool qk8, int n_cu)
{
    return std::max(prefill_workspace_min(p, d, block_kv, causal, n_cu),
                    make_plan(p, d, block_kv, causal, qk8, n_cu, ~(size_t)0).bytes);
}

// A split over the keys runs over as many workgroups as the caller's workspace
// has room for; without one the tiles run unsplit (same codes and counts).
hipError_t launch_prefill(const Params& p_in, int d, int block_kv, bool causal, bool count, int scale,
                          bool qk8, int n_cu, void* ws, size_t ws_bytes, hipStream_t stream)
{
    Params p = p_in;
    p.causal = causal;
    p.ws_max = nullptr;
    p.ws_part = nullptr;
    const Plan pl = make_plan(p, d, block_kv, causal, qk8, n_cu, ws ? ws_bytes : 0);
    const long long per_unit = pl.C * pl.cols;
    const long long slots = (pl.units + kNumXcd - 1) / kNumXcd * per_unit;
    if (slots * kNumXcd > 1 << 30)
        return hipErrorInvalidValue;
    p.n_tiles = (int)pl.tiles;
    p.run = (int)pl.run;
    p.run_tiles = (int)((pl.run + pl.rows - 1) / pl.rows);
    p.nsplit = (int)pl.C;
    p.total_wg = (int)(pl.units * per_unit);
    p.per_xcd = (int)slots;
    if (pl.C == 1)
        return launch_phase(p, pl, d, block_kv, count, scale, qk8, 0, stream);
    p.ws_max = static_cast<float*>(ws);
    p.ws_part = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + pl.off_part);
    if (count)
        hipLaunchKernelGGL(prefill_zero, dim3(1024), dim3(256), 0, stream, p.counts,
                           (int64_t)p.B * p.Hq * p.N * 3);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = launch_phase(p, pl, d, block_kv, count, scale, qk8, 1, stream);
    if (e == hipSuccess)
        e = launch_phase(p, pl, d, block_kv, count, scale, qk8, 2, stream);
    if (e == hipSuccess) {
        const dim3 grid((unsigned)(pl.units * pl.rows));
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, p); };
        if (pl.rows == 16)
            d == 64 ? go(prefill_merge<64, 16>) : go(prefill_merge<128, 16>);
        else
            d == 64 ? go(prefill_merge<64, 32>) : go(prefill_merge<128, 32>);
        e = hipGetLastError();
    }
    return e;
}

int prefill_rows_per_wg() { return 32; }

}  // namespace attn
