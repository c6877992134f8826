// Launch of the KV-cache kernel (attn_prefill_kernel.hpp) by its plan
// (attn_plan.hpp), and the merge of a split tile.
#include "attn_common.hpp"
#include "attn_launch.hpp"

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

hipError_t launch_phase(const Params& p, const KvPlan& pl, int d, int block_kv, bool count, int scale, bool qk8,
                        int phase, hipStream_t s)
{
    auto go = [&](auto fn) { return fn(p, d, block_kv, count, scale, phase, pl.cols, pl.waves, s); };
    if (pl.rows == 16)
        return qk8 ? go(launch_kv_t<true, 16>) : go(launch_kv_t<false, 16>);
    return qk8 ? go(launch_kv_t<true, 32>) : go(launch_kv_t<false, 32>);
}

}  // namespace

hipError_t launch_prefill(const Params& p_in, const KvPlan& pl, int d, int block_kv, bool causal, bool count,
                          int scale, bool qk8, void* ws, hipStream_t stream)
{
    Params p = p_in;
    p.causal = causal;
    p.ws_max = nullptr;
    p.ws_part = nullptr;
    const long long per_unit = pl.C * pl.cols;
    if (pl.slots * kNumXcd > 1 << 30)
        return hipErrorInvalidValue;
    p.n_tiles = (int)pl.tiles;
    p.run = (int)pl.run;
    p.run_tiles = (int)((pl.run + pl.rows - 1) / pl.rows);
    p.nsplit = (int)pl.C;
    p.total_wg = (int)(pl.units * per_unit);
    p.per_xcd = (int)pl.slots;
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

}  // namespace attn
