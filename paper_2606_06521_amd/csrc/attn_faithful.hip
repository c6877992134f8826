// Faithful mode: FP32 Q, K, V; only P is rounded to E4M3 values (Sec. 6.1:
// Q, K, V stay in FP32 so that the P-cast is the only quantisation).
//
// Algorithm 1 per query row.  Scores and the P.V product run on the FP32 MFMA;
// exp2 is evaluated in FP64 and rounded once to FP32; P*S goes through the
// hardware E4M3 convert (round to nearest even) and straight back through the
// hardware decode, so the P.V operand holds the exact E4M3 values.
// ATTN_MODE_NOCAST (CAST = false) skips the convert.  DYN: the dynamic
// per-block power-of-two scale (the cast of each block uses 2^kj instead of S).
//
// A workgroup holds TR query rows (32 or 16); its NW waves take the KV blocks
// of the visit in rounds, wave w the block at visit position NW i + w of round
// i.  Each wave takes the row maxima of its block's scores and puts them in
// LDS; after the round's one barrier the running maximum the sequential visit
// has reached at that block is the maximum over the earlier rounds (carried by
// every wave) and the waves below w.  Every block therefore sees exactly the
// running maximum of Algorithm 1: P, its E4M3 code and the counts are those of
// the one-wave visit.  Each wave keeps its own (O, l); at the end they are
// brought to the rows' final maximum and summed in a fixed order, so only the
// FP32 rounding of O and l depends on the split.
//
// K and V go from memory straight into the MFMA operands: the FP32 MFMA
// takes 64 cycles per 2 x 32 x 32 (32 per 4 x 16 x 16), so one 16-byte load
// per lane feeds four of them and a ring of loads in flight covers the
// latency; staging through LDS would only add barriers.  They are buffer
// loads: keys past the end read 0 without a clamp, and an address costs no
// vector instruction.  The k index of the scores' MFMA is a permutation of d
// under which a row's load is contiguous across the lane groups, and the M
// index of P.V one of d under which a lane loads 16 contiguous bytes of V.
//
// What bounds it: the FP32 MFMA and the vector instructions do not overlap on
// a SIMD (without its exp2s the kernel is shorter by their whole issue time,
// without its loads by 4 %), so the vector work per key is kept low: exp2 in
// 18 instructions, the power-of-two scale inside the convert, no rescale of O
// while no row's maximum moves, no address arithmetic.
// Measured (four waves of 32 rows staging K and V through LDS, then this):
// 8 heads x 4096 x 4096, d = 128: 806 -> 543 us, 85 -> 126 TFLOP/s of the 154 a
// large FP32 matrix product reaches; 64 x (32 queries x 4096 keys), d = 128:
// 924 -> 85 us; 1024 x 1024, d = 64: 114 -> 16 us.
#include "attn_common.hpp"
#include "attn_launch.hpp"

#include <math.h>
#include <type_traits>

namespace attn {

namespace {

// The FP32 MFMA of a TR-row tile.  Lane (n, g): query row n of the tile,
// group g of NG.  S^T tile of TR keys: register r of group g holds key
// KPG g + r (A row n is key a_key(n)).
template <int TR>
struct Tile;

template <>
struct Tile<32> {
    static constexpr int NG = 2, KPG = 16;
    using Acc = f32x16;
    static __device__ inline Acc mma(float a, float b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int a_key(int n) { return a_row_to_key(n); }
    // M index of accumulator register r
    static __device__ inline int d_row(int r, int g) { return 8 * (r / 4) + 4 * g + (r % 4); }
};

template <>
struct Tile<16> {
    static constexpr int NG = 4, KPG = 4;
    using Acc = f32x4;
    static __device__ inline Acc mma(float a, float b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int a_key(int n) { return n; }
    static __device__ inline int d_row(int r, int g) { return 4 * g + r; }
};

// combine over the lane groups holding one row
template <int NG, typename T, typename F>
__device__ inline T over_groups(T x, F f)
{
#pragma unroll
    for (int off = 64 / NG; off < 64; off <<= 1)
        x = f(x, __shfl_xor(x, off, 64));
    return x;
}

template <int N>
using vecf = __attribute__((__vector_size__(N * sizeof(float)))) float;

}  // namespace

template <int D, int BC, bool COUNT, bool CAST, int SCALE, int TR, int NW, int DS>
__global__ void __launch_bounds__(64 * NW, 2) faithful_kernel(Params p)
{
    using TL = Tile<TR>;
    using Acc = typename TL::Acc;
    constexpr int NG = TL::NG;            // lane groups (k indices per MFMA)
    constexpr int KPG = TL::KPG;          // keys per group and tile (accumulator registers)
    constexpr int KT = BC / TR;           // S^T tiles per KV block
    constexpr int DQ = D / (4 * NG);      // 16-byte pieces of a Q / K row per lane
    constexpr int DO = D / DS;            // columns of O in this workgroup
    constexpr int DT = DO / TR;           // d tiles of O^T
    constexpr int VW = DT < 4 ? DT : 4;   // floats per V load; tile (t, e) row m is column VW TR t + VW m + e
    constexpr int VT = DT / VW;           // V loads per key
    constexpr int MS = DO + 4;            // padded row stride of the merge buffer (floats)
    constexpr int QS = D + 4;             // ... of the Q rows
    constexpr int ROW = 4 * D;            // bytes of a K / V row
    constexpr int NK = KT * DQ;           // K loads of a block
    constexpr int NV = KT * KPG * VT;     // V loads of a block
    // loads in flight; a 16-row tile has the registers to request the next
    // phase's first loads before the barrier and before P.V
    constexpr bool AHEAD = TR == 16;
    constexpr int PFK = AHEAD && NK >= 16 ? 16 : 8;
    constexpr int PFV = AHEAD && NV >= 16 ? 16 : 8;
    static_assert(NK % 4 == 0 && NK >= PFK && NV >= PFV && NW * MS >= QS, "ring and buffer sizes");
    using V4 = vecf<4>;
    using VV = vecf<VW>;

    // the tile's Q rows during the visit, then every wave's O for the merge
    __shared__ __attribute__((aligned(16))) float mbuf[NW * TR * MS];
    __shared__ float tab[2][NW][TR];      // row maxima of the round's blocks
    __shared__ float lsh[NW][TR];
    __shared__ uint32_t csh[TR][3];

    int bh, tile;
    if (!(p.causal ? map_tile<true>(p, bh, tile) : map_tile<false>(p, bh, tile)))
        return;
    const int part = DS == 1 ? 0 : bh % DS;       // which columns of O (DS workgroups per tile)
    bh /= DS;
    const int N = p.N, Nk = p.Nk, qoff = p.qoff;   // query rows, keys, row r at key r + qoff
    const bool causal = p.causal != 0;
    const int b = bh / p.Hq;
    const int hq = bh - b * p.Hq;
    const int hk = hq / (p.Hq / p.Hkv);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & (TR - 1);        // query row within the tile (also the MFMA A row)
    const int g = lane / TR;              // lane group
    const int row0 = tile * TR;
    const int row = row0 + n;

    const float* Qg = static_cast<const float*>(p.q) + (size_t)bh * N * D;
    const size_t kvoff = ((size_t)b * p.Hkv + hk) * (size_t)Nk * D;
    const float* Kg = static_cast<const float*>(p.k) + kvoff;
    const float* Vg = static_cast<const float*>(p.v) + kvoff;

    // blocks the tile visits
    const int rlast = min(row0 + TR, N) - 1;
    const int nbt = causal ? (rlast + qoff) / BC + 1 : (Nk + BC - 1) / BC;
    auto jof = [&](int it) __attribute__((always_inline)) { return p.order == 0 ? it : nbt - 1 - it; };

    // K piece i of a block: tile i / DQ, piece i % DQ of row a_key
    const int k_lane = TL::a_key(n) * ROW + 16 * g;
    auto kload = [&](__amdgpu_buffer_rsrc_t kb, int i) __attribute__((always_inline)) {
        return __builtin_bit_cast(V4, __builtin_amdgcn_raw_buffer_load_b128(kb, k_lane + 16 * NG * (i % DQ),
                                                                           TR * (i / DQ) * ROW, 0));
    };
    // V piece i of a block: key (i / VT) of the group's keys, piece i % VT of the row
    const int v_lane = KPG * g * ROW + 4 * VW * n + 4 * DO * part;
    auto vload = [&](__amdgpu_buffer_rsrc_t vb, int i) __attribute__((always_inline)) {
        const int kr = i / VT;
        const int so = (TR * (kr / KPG) + kr % KPG) * ROW;
        if constexpr (VW == 4)
            return __builtin_bit_cast(VV, __builtin_amdgcn_raw_buffer_load_b128(vb, v_lane + 4 * VW * TR * (i % VT), so, 0));
        else if constexpr (VW == 2)
            return __builtin_bit_cast(VV, __builtin_amdgcn_raw_buffer_load_b64(vb, v_lane + 4 * VW * TR * (i % VT), so, 0));
        else
            return __builtin_bit_cast(VV, __builtin_amdgcn_raw_buffer_load_b32(vb, v_lane + 4 * VW * TR * (i % VT), so, 0));
    };
    auto kbuf = [&](int t0) __attribute__((always_inline)) { return row_buffer(Kg + (size_t)t0 * D, (size_t)(Nk - t0) * ROW); };
    auto vbuf = [&](int t0) __attribute__((always_inline)) { return row_buffer(Vg + (size_t)t0 * D, (size_t)(Nk - t0) * ROW); };

    V4 ka[PFK];
    VV va[PFV];
    if (AHEAD && w < nbt) {
        const auto kb = kbuf(jof(w) * BC);
#pragma unroll
        for (int i = 0; i < PFK; ++i)
            ka[i] = kload(kb, i);
    }

    if (COUNT && tid < TR * 3)
        csh[tid / 3][tid % 3] = 0u;
    // Q^T fragments: lane (n, g) takes Q[row][4 NG i + 4 g .. +4] from LDS (in
    // registers they would cost DQ * 4 of the 256; one read feeds four MFMAs)
    for (int e = tid; e < TR * D / 4; e += 64 * NW) {
        const int rr = e / (D / 4), piece = e % (D / 4);
        *reinterpret_cast<V4*>(mbuf + rr * QS + 4 * piece) =
            row0 + rr < N ? *reinterpret_cast<const V4*>(Qg + (size_t)(row0 + rr) * D + 4 * piece) : V4{};
    }
    const float* const q_lane = mbuf + n * QS + 4 * g;
    lds_barrier();

    const float c = p.c;
    const float S = p.S;
    float carry = -INFINITY;          // the rows' running maximum after the earlier rounds
    float m_run = -INFINITY;          // ... after this wave's last block
    float mc_run = -INFINITY;
    float ell = 0.f;                  // partial sum of this lane group
    Acc o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        o[dt] = Acc{};
    uint32_t cnt0 = 0, cnt1 = 0, cnt2 = 0;

    const int rounds = (nbt + NW - 1) / NW;
    for (int rd = 0; rd < rounds; ++rd) {
        const int it = rd * NW + w;
        const bool on = it < nbt;
        const int j = jof(it);
        const int t0 = j * BC;
        Acc s[KT];
        float mx = -INFINITY;
        if (on) {
            // ---- S^T = K_j Q^T (raw dot products) ----
            const auto kb = kbuf(t0);
            auto qload = [&](int i) __attribute__((always_inline)) {
                return *reinterpret_cast<const V4*>(q_lane + 4 * NG * (i % DQ));
            };
            V4 qn = qload(0);
            if (!AHEAD) {
#pragma unroll
                for (int i = 0; i < PFK; ++i)
                    ka[i] = kload(kb, i);
            }
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const int kt = i / DQ;
                const V4 cur = ka[i % PFK], q4 = qn;
                if (i + 1 < NK)
                    qn = qload(i + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    s[kt] = TL::mma(cur[e], q4[e], i % DQ == 0 && e == 0 ? Acc{} : s[kt]);
                // a row's next 128 bytes are requested together: their pieces
                // then share the cache line while it is on its way
                if (i % 4 == 3 && i + PFK - 3 < NK) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        ka[(i - 3 + u) % PFK] = kload(kb, i - 3 + u + PFK);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (AHEAD) {
                const auto vb = vbuf(t0);
#pragma unroll
                for (int i = 0; i < PFV; ++i)
                    va[i] = vload(vb, i);
                __builtin_amdgcn_sched_barrier(0);
            }

            // ---- mask: keys past the sequence end, keys after the row (causal) ----
            if ((causal && t0 + BC - 1 > row0 + qoff) || t0 + BC > Nk) {
                const int lim = (causal ? min(row + qoff, Nk - 1) : Nk - 1) - t0 - KPG * g;
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < KPG; ++r)
                        if (TR * kt + r > lim)
                            s[kt][r] = -INFINITY;
            }
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < KPG; ++r)
                    mx = fmax_f(mx, s[kt][r]);
            mx = over_groups<NG>(mx, [](float x, float y) { return fmax_f(x, y); });
        }
        // ---- the running maximum before this block ----
        float(*const tb)[TR] = tab[rd & 1];
        if (g == 0)
            tb[w][n] = mx;
        lds_barrier();
        float m_prev = carry;
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            const float t = tb[v][n];
            if (v < w)
                m_prev = fmax_f(m_prev, t);
            carry = fmax_f(carry, t);
        }
        if (!on)
            continue;

        // ---- m_new = max(m, max Z); alpha = exp(m - m_new) (base 2) ----
        const bool vis = mx > -INFINITY;            // the row has a key in this block
        const float m_new = fmax_f(m_prev, mx);
        const float mc_new = m_new * c;
        // before the row's first valid key (possible only with qoff > 0 in
        // reverse order) nothing has accumulated: alpha is irrelevant and P
        // must be 0 (x = -inf), not NaN
        const bool none = mc_new == -INFINITY;
        const float alpha = none ? 1.f : exp2_f64(mc_run - mc_new);
        const float nmc = none ? 0.f : -mc_new;
        if (COUNT && part == 0 && p.gap_hist && vis && g == 0 && row < N)
            record_gap(p, bh, j, mx, c, nmc);
        // Dynamic P-scale: this block's rows cast P * 2^kj, kj = k0 +
        // clamp(floor(-xmax), 0, 126 - k0) with xmax = fma(block max, c, -mc),
        // and the decoded value goes back to S units times 2^(k0 - kj) (exact)
        float cvt_scale = p.inv_S, back = 1.f;
        if constexpr (SCALE == kScaleDynamic) {
            const float xmax = __builtin_fmaf(mx, c, nmc);
            const float f = __builtin_fminf(__builtin_fmaxf(__builtin_floorf(-xmax), 0.f), (float)(126 - p.k0));
            const int kj = p.k0 + (int)f;
            cvt_scale = __uint_as_float((uint32_t)(127 - kj) << 23);
            back = __uint_as_float((uint32_t)(127 + p.k0 - kj) << 23);
        }

        // ---- P = exp(Z - m_new); l from pre-cast P; P~ = E4M3(P*S), in place ----
        float lsum = 0.f;
        uint32_t bz = 0;   // zero codes of this block (valid rows and keys)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
            for (int r = 0; r < KPG; r += 2) {
                const float p0 = exp2_f64(__builtin_fmaf(s[kt][r], c, nmc));
                const float p1 = exp2_f64(__builtin_fmaf(s[kt][r + 1], c, nmc));
                lsum += p0;
                lsum += p1;
                float y0, y1;
                if constexpr (CAST) {
                    int code;
                    if constexpr (SCALE == kScaleAny) {
                        // saturate at the largest finite E4M3 value before the convert
                        code = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_fminf(p0 * S, 448.f),
                                                               __builtin_fminf(p1 * S, 448.f), 0, false);
                    } else {
                        code = __builtin_bit_cast(
                            int, __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(s16x2{}, p0, p1, cvt_scale, false));
                    }
                    if (COUNT) {
                        const int k0 = t0 + TR * kt + KPG * g + r;
                        const bool z0 = (code & 0xFF) == 0 && k0 < Nk && (!causal || k0 <= row + qoff);
                        const bool z1 = (code & 0xFF00) == 0 && k0 + 1 < Nk && (!causal || k0 + 1 <= row + qoff);
                        if (j > 0) {
                            cnt2 += z0 + z1;
                        } else {
                            if (z0) { if (k0 < p.n_sink) ++cnt0; else ++cnt1; }
                            if (z1) { if (k0 + 1 < p.n_sink) ++cnt0; else ++cnt1; }
                        }
                        if (row < N)
                            bz += z0 + z1;
                    }
                    const auto dec = __builtin_amdgcn_cvt_pk_f32_fp8(code, false);
                    y0 = dec[0];
                    y1 = dec[1];
                    if constexpr (SCALE == kScaleDynamic) {
                        y0 *= back;
                        y1 *= back;
                    }
                } else {
                    y0 = p0 * S;
                    y1 = p1 * S;
                }
                s[kt][r] = y0;
                s[kt][r + 1] = y1;
                if (COUNT && r % 4 == 2)
                    __builtin_amdgcn_sched_barrier(0);   // keeps the counts' temporaries few
            }
        }
        ell = alpha * ell + lsum;
        if (COUNT && CAST && part == 0 && p.blk_zero)
            record_block_zeros(p, bh, j, bz);

        // ---- O <- alpha O + P~ V_j  (FP32 MFMA on O^T = V^T P~^T) ----
        // (alpha is exactly 1 in every lane while no row's maximum moves)
        if (__ballot(alpha != 1.0f) != 0) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < KPG; ++r)
                    o[dt][r] *= alpha;
        }
        if (AHEAD && it + NW < nbt) {
            const auto kb = kbuf(jof(it + NW) * BC);
#pragma unroll
            for (int i = 0; i < PFK; ++i)
                ka[i] = kload(kb, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        {
            const auto vb = vbuf(t0);
            if (!AHEAD) {
#pragma unroll
                for (int i = 0; i < PFV; ++i)
                    va[i] = vload(vb, i);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int kr = i / VT;
                const VV cur = va[i % PFV];
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    o[VW * (i % VT) + e] = TL::mma(cur[e], s[kr / KPG][kr % KPG], o[VW * (i % VT) + e]);
                if (i + PFV < NV)
                    va[i % PFV] = vload(vb, i + PFV);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        m_run = m_new;
        mc_run = mc_new;
    }

    // ---- merge: each wave's (O, l) at the rows' final maximum, summed in wave order ----
    const float mc_final = carry * c;
    const float beta = mc_run == mc_final ? 1.f : mc_run == -INFINITY ? 0.f : exp2_f64(mc_run - mc_final);
    const float ell_w = over_groups<NG>(ell, [](float x, float y) { return x + y; }) * beta;
    lds_barrier();                        // the last Q reads
    float* const mw = mbuf + (w * TR + n) * MS;
#pragma unroll
    for (int t = 0; t < VT; ++t)
#pragma unroll
        for (int r = 0; r < KPG; ++r) {
            VV x;
#pragma unroll
            for (int e = 0; e < VW; ++e)
                x[e] = o[VW * t + e][r] * beta;
            *reinterpret_cast<VV*>(mw + VW * TR * t + VW * TL::d_row(r, g)) = x;
        }
    if (COUNT) {
        auto add = [](uint32_t x, uint32_t y) { return x + y; };
        cnt0 = over_groups<NG>(cnt0, add);
        cnt1 = over_groups<NG>(cnt1, add);
        cnt2 = over_groups<NG>(cnt2, add);
    }
    if (g == 0) {
        lsh[w][n] = ell_w;
        if (COUNT) {
            atomicAdd(&csh[n][0], cnt0);
            atomicAdd(&csh[n][1], cnt1);
            atomicAdd(&csh[n][2], cnt2);
        }
    }
    __syncthreads();
    if (p.out) {
        for (int e = tid; e < TR * DO / 4; e += 64 * NW) {
            const int rr = e / (DO / 4), piece = e % (DO / 4);
            if (row0 + rr >= N)
                continue;
            V4 acc{};
            float l = 0.f;
#pragma unroll
            for (int v = 0; v < NW; ++v) {
                acc += *reinterpret_cast<const V4*>(mbuf + (v * TR + rr) * MS + 4 * piece);
                l += lsh[v][rr];
            }
            const float denom = S * l;
            V4 v4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v4[i] = acc[i] / denom * p.v_descale;
            *reinterpret_cast<V4*>(p.out + ((size_t)bh * N + row0 + rr) * D + DO * part + 4 * piece) = v4;
        }
    }
    if (part == 0 && tid < TR && row < N) {      // lane tid of wave 0 holds row tid (group 0)
        const size_t flat = (size_t)bh * N + row;
        float l = 0.f;
#pragma unroll
        for (int v = 0; v < NW; ++v)
            l += lsh[v][tid];
        if (p.lse)
            p.lse[flat] = (float)(((double)mc_final + log2((double)l)) * 0.6931471805599453094);
        if (COUNT) {
            p.counts[3 * flat + 0] = csh[tid][0];
            p.counts[3 * flat + 1] = csh[tid][1];
            p.counts[3 * flat + 2] = csh[tid][2];
        }
    }
}

namespace {

template <int D, int BC, bool COUNT, bool CAST, int SCALE, int TR, int NW, int DS>
hipError_t launch_one(const Params& p_in, hipStream_t stream)
{
    Params p = p_in;
    p.n_tiles = (p.N + TR - 1) / TR;
    const long long total = (long long)p.B * p.Hq * DS * p.n_tiles;
    if (total > 1 << 30)
        return hipErrorInvalidValue;
    p.total_wg = (int)total;
    p.per_xcd = (p.total_wg + kNumXcd - 1) / kNumXcd;
    hipLaunchKernelGGL((faithful_kernel<D, BC, COUNT, CAST, SCALE, TR, NW, DS>), dim3(p.per_xcd * kNumXcd),
                       dim3(64 * NW), 0, stream, p);
    return hipGetLastError();
}

// Tile and workgroup shape by how far the 32-row tiles fill the chip:
// - two workgroups of four waves per CU when there are enough of them (the two
//   drift apart, so one's loads and barriers fall into the other's MFMAs);
// - one of eight waves, when every CU still gets one;
// - 16-row tiles below that, and up to one per two CUs each of them by two
//   workgroups that compute the same scores and half of the columns of O:
//   three quarters of the tile's work on each, on CUs that would idle
//   (64 x (32 x 4096), 128 tiles: 118 us with one workgroup per tile, 85 with
//   two and the loads requested ahead).
template <int D, int BC, bool COUNT, bool CAST, int SCALE>
hipError_t launch_shape(const Params& p, int n_cu, hipStream_t s)
{
    const long long heads = (long long)p.B * p.Hq;
    const long long tiles32 = heads * ((p.N + 31) / 32), tiles16 = heads * ((p.N + 15) / 16);
    if (tiles32 >= 2LL * n_cu)
        return launch_one<D, BC, COUNT, CAST, SCALE, 32, 4, 1>(p, s);
    if (tiles32 >= n_cu)
        return launch_one<D, BC, COUNT, CAST, SCALE, 32, 8, 1>(p, s);
    if (2 * tiles16 > n_cu)
        return launch_one<D, BC, COUNT, CAST, SCALE, 16, 8, 1>(p, s);
    return launch_one<D, BC, COUNT, CAST, SCALE, 16, 8, 2>(p, s);
}

// Without the cast the dynamic scale is the static one (P * 2^kj * 2^(k0-kj)
// = P * S exactly), so ATTN_MODE_NOCAST ignores it.
template <int D, int BC, bool COUNT>
hipError_t launch_cast(const Params& p, bool cast, int scale, int n_cu, hipStream_t s)
{
    if (!cast)
        return launch_shape<D, BC, COUNT, false, kScaleAny>(p, n_cu, s);
    if (scale == kScaleDynamic)
        return launch_shape<D, BC, COUNT, true, kScaleDynamic>(p, n_cu, s);
    if (scale == kScalePow2)
        return launch_shape<D, BC, COUNT, true, kScalePow2>(p, n_cu, s);
    return launch_shape<D, BC, COUNT, true, kScaleAny>(p, n_cu, s);
}

template <int D, int BC>
hipError_t launch_d_bc(const Params& p, bool count, bool cast, int scale, int n_cu, hipStream_t s)
{
    return count ? launch_cast<D, BC, true>(p, cast, scale, n_cu, s)
                 : launch_cast<D, BC, false>(p, cast, scale, n_cu, s);
}

}  // namespace

hipError_t launch_faithful(const Params& p_in, int d, int block_kv, bool causal, bool count, bool cast,
                           int scale, int n_cu, hipStream_t stream)
{
    Params p = p_in;
    p.causal = causal;
    if (d == 64)
        return block_kv == 64 ? launch_d_bc<64, 64>(p, count, cast, scale, n_cu, stream)
                              : launch_d_bc<64, 128>(p, count, cast, scale, n_cu, stream);
    return block_kv == 64 ? launch_d_bc<128, 64>(p, count, cast, scale, n_cu, stream)
                          : launch_d_bc<128, 128>(p, count, cast, scale, n_cu, stream);
}

}  // namespace attn
