// KV-cache kernel (fast modes): few query rows per (batch, KV head) against Nk
// cached keys -- decode, short chunks, and the shape of the paper's Exp. 1
// (q_len = 32 against N = 4096).  Query row r sits at key position
// Nk - Nq + r (causal rows see keys up to their position).
//
// The query heads of a group read the same keys, so their rows are one run of
// G * Nq rows (contiguous in q, out, lse and counts: row R is query R % Nq of
// head R / Nq) cut into tiles of TR = 16 or 32 rows: a decode step with four
// query heads per KV head reads each key once instead of four times.  Causal
// heads of 128 rows or more get tiles of their own: every row of a tile meets
// the V of all blocks the tile visits (with P = 0 where masked, but 0 times NaN
// is NaN), and a tile that holds the end of one head and the start of the next
// visits them all.  Its rows would also be masked in most of them.
//
// A tile's workgroup has NW = 8 or 4 waves.  They take the KV blocks of the visit
// in rounds, wave w the block at visit position NW i + w of round i.  Each wave
// takes the row maxima of its block's scores and puts them in LDS; after the
// round's one barrier the running maximum the sequential visit has reached at
// that block is the maximum over the earlier rounds (carried by every wave)
// and the waves below w.  Every block sees exactly the running maximum of
// Algorithm 1, so P = exp2(fma(D, c, -mc)), its E4M3 code and the counts are
// those of the one-wave visit, and K is read once.  Each wave keeps its own
// (O, l); at the end they are brought to the rows' final maximum and summed in
// a fixed order: only the FP32 rounding of O and l depends on the split.
//
// When the tiles alone cannot fill the chip, a tile's visit is cut into
// nsplit contiguous ranges, one workgroup each, and the work becomes three
// launches on the stream:
//   PHASE 1: every workgroup writes the row maxima of its range to the workspace;
//   PHASE 2: the rounds above over its range, starting from the maximum over
//            the earlier ranges; (O, l) at the tile's final maximum go to the
//            workspace;
//   merge:   the nsplit partial sums are added in a fixed order.
// The launch boundaries order the phases; no workgroup waits on another.  This
// reads K twice.  PHASE 0 is the one-workgroup kernel; DS = 2 of them share a
// tile when that fills CUs that would idle: both compute the scores (K comes
// from their XCD's L2 the second time), each takes half of the columns of V.
//
// K and V come by buffer loads (keys past the end read 0 and are masked).  K
// goes through registers (a ring of tiles in flight) and a 2 KB LDS buffer per
// wave: fetching the MFMA's A operand straight from memory, 16 rows per 16
// lanes, costs the CU's cache one lookup per lane and caps it at 16 B per
// cycle.  The V block goes straight into the wave's LDS stage (no registers)
// in the XOR-swizzled layout read transposed by ds_read_b64_tr_b8.
//
// What bounds it: the stream of K and V where the cache is long (decode of 16
// requests x 32/8 heads x 8192 keys: 403 MB in 81 us, 5.0 TB/s), the softmax of a
// block per wave where a group has many rows, and 8 to 10 us of launch, first
// round trip and merge on short visits.  Measured against one 32-row tile per
// query head that read K twice (inputs that change from call to call): that
// decode 263 -> 81 us; one request x 131001 E4M3 keys 155 -> 74; 64 x (32
// queries x 4096 keys) 41 -> 33.
#pragma once

#include "attn_common.hpp"
#include "attn_launch.hpp"

#include <math.h>
#include <type_traits>

namespace attn {

namespace {

__device__ inline i32x2 read_tr8(const uint8_t* p)
{
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)(p));
}

// The MFMA shapes of a TR-row tile.  Lane (n, g): row n, group g of NG.
//   TR = 32: S^T by 32x32x16 bf16 / 32x32x64 E4M3, P.V by 32x32x64 E4M3
//   TR = 16: S^T by 16x16x32 bf16 / 16x16x128 E4M3, P.V by 16x16x128 E4M3
// The keys of an S^T tile are chosen so that a lane's E4M3 bytes are the B
// operand of P.V as they stand, in runs of eight consecutive keys (the unit
// in which the FP8 matrix core aligns products):
//   TR = 32: register r of tile kt, group g: key 32 kt + 16 g + r
//   TR = 16:                                 key (BC / 4) g + 4 kt + r
template <int TR, int BC>
struct KvTile;

template <int BC>
struct KvTile<32, BC> {
    static constexpr int NG = 2, REGS = 16, TSTEP = 32, GSTEP = 16;
    using Acc = f32x16;
    static __device__ inline int a_key(int n) { return a_row_to_key(n); }
    static __device__ inline int d_row(int r, int g) { return 8 * (r / 4) + 4 * g + (r % 4); }
    static __device__ inline Acc qk16(bf16x8 a, bf16x8 b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
    template <bool SCALED>
    static __device__ inline Acc f8(i32x8 a, i32x8 b, Acc c, int sb)
    {
        return SCALED ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, sb)
                      : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
    }
};

template <int BC>
struct KvTile<16, BC> {
    static constexpr int NG = 4, REGS = 4, TSTEP = 4, GSTEP = BC / 4;
    using Acc = f32x4;
    static __device__ inline int a_key(int n) { return GSTEP * (n >> 2) + (n & 3); }
    static __device__ inline int d_row(int r, int g) { return 4 * g + r; }
    static __device__ inline Acc qk16(bf16x8 a, bf16x8 b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
    template <bool SCALED>
    static __device__ inline Acc f8(i32x8 a, i32x8 b, Acc c, int sb)
    {
        return SCALED ? __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, sb)
                      : __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
    }
};

}  // namespace

template <int D, int BC, bool COUNT, int SCALE, bool QK8, int TR, int PHASE, int DS, int NW>
__global__ void __launch_bounds__(64 * NW, 2) kv_kernel(Params p)
{
    using TL = KvTile<TR, BC>;
    using Acc = typename TL::Acc;
    constexpr int NG = TL::NG, REGS = TL::REGS;
    constexpr int KT = BC / TR;                 // S^T tiles per block
    constexpr int DO = D / DS;                  // columns of O in this workgroup
    constexpr int DT = DO / TR;                 // d tiles of O^T
    constexpr int KROW = QK8 ? D : 2 * D;       // bytes per Q / K row
    constexpr int VROW = DO;                    // bytes of a V row in this workgroup
    // 16-byte pieces of a row per lane; a k-step takes one (bf16) or two (E4M3;
    // one and zeros where a row of 64 bytes is half of the k-step)
    constexpr int NP = KROW / (16 * NG);
    constexpr int PPS = QK8 ? (NP >= 2 ? 2 : 1) : 1;
    constexpr int DK = NP / PPS;                // k-steps
    constexpr int KSB = 16 * PPS * NG;          // bytes of a row per k-step
    // K goes through registers and a small LDS buffer per wave, one segment of
    // SEG bytes of a tile's rows at a time
    constexpr int SEG = KROW < 128 ? KROW : (TR == 16 ? 128 : 64);
    constexpr int NSEG = KROW / SEG;
    constexpr int IPS = TR * SEG / 1024;        // load instructions per segment
    constexpr int SCH = SEG / 16;               // chunks per row of a segment
    constexpr int SPS = SEG / (KSB < SEG ? KSB : SEG);   // k-steps per segment
    constexpr int KB_BYTES = TR * SEG;          // the wave's K buffer
    // K tiles in flight: 64 registers of a 16-row tile, 32 of a 32-row one (a CU
    // streams at its full rate with 32 KB in flight, a quarter of either)
    constexpr int KREGS = TR == 16 ? 64 : 32;
    constexpr int RING = KT * NP * 4 <= KREGS ? KT : KREGS / (NP * 4);
    constexpr int VCPR = VROW / 16;             // 16-byte chunks per V row
    constexpr int V_BYTES = BC * VROW;          // one wave's V stage
    constexpr int V_NI = V_BYTES / 1024;        // 16-byte-per-lane rounds per stage
    constexpr int V_RPI = 1024 / VROW;          // V rows per round
    constexpr int PW = KT * REGS / 4;           // words of E4M3 bytes per lane
    constexpr int PVS = PW > 8 ? PW / 8 : 1;    // P.V k-steps (32 bytes per lane; with BC = 64, TR = 16 half zeros)
    constexpr int MS = DO + 4;                  // padded row stride of the merge buffer (floats)
    constexpr int MERGE_BYTES = NW * TR * MS * 4;
    constexpr int KB_OFF = PHASE == 1 ? 0 : NW * V_BYTES;
    constexpr int LDS_BYTES = KB_OFF + NW * KB_BYTES > MERGE_BYTES || PHASE == 1 ? KB_OFF + NW * KB_BYTES : MERGE_BYTES;
    static_assert(DS == 1 || PHASE == 0, "the split in columns is unsplit in keys");
    static_assert(RING >= 1 && KT % RING == 0 && NSEG * IPS == NP && NSEG * SPS == DK, "K ring and segments");

    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    __shared__ float tab[2][NW][TR];            // row maxima of the round's blocks
    __shared__ float lsh[NW][TR];               // merge: each wave's l, at the final maximum
    __shared__ uint32_t csh[TR][3];             // merge: counts
    __shared__ float rmax[PHASE == 2 ? 64 * NW : 1];   // PHASE 2: the maxima of every range

    // workgroup -> (tile unit, range cidx of C).  Logical indices run over (batch,
    // KV head), range, tile, and each XCD takes a contiguous run of per_xcd of
    // them: the tiles that read a range's keys share an L2, and no XCD gets more
    // workgroups than another (the ranges of a tile share nothing).
    const int C = PHASE == 0 ? 1 : p.nsplit;
    int unit, cidx;
    {
        const int i = blockIdx.x;
        const int slot = i / kNumXcd;
        if (slot >= p.per_xcd)
            return;
        const int L = (i % kNumXcd) * p.per_xcd + slot;
        if (L >= p.total_wg)
            return;
        const int per_range = DS * p.n_tiles;
        const int range = L / per_range;
        const int head = range / C;
        cidx = range - head * C;
        unit = head * per_range + L - range * per_range;
    }
    // DS workgroups per tile: the same scores, DO columns of V and O each
    const int colp = DS == 1 ? 0 : unit % DS;
    unit /= DS;
    const int bk = unit / p.n_tiles;            // (batch, KV head)
    // (causal: the tiles with the most blocks start first)
    const int tile = p.causal ? p.n_tiles - 1 - (unit - bk * p.n_tiles) : unit - bk * p.n_tiles;
    const int Nq = p.N, Nk = p.Nk, qoff = p.qoff;
    const bool causal = p.causal != 0;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & (TR - 1);
    const int g = lane / TR;
    // rows of the group share tiles in runs: the whole group's, or one head's
    const int run = tile / p.run_tiles;
    const int rows = (run + 1) * p.run;         // end of the tile's run
    const int row0 = run * p.run + TR * (tile - run * p.run_tiles);
    const int row = row0 + n;                   // every wave holds the same TR rows
    const int q0 = row0 % Nq;                   // the tile's first query position
    const int pos = (q0 + n) % Nq + qoff;       // the row's key position
    const int nrow = min(TR, rows - row0);
    const int pos_min = (q0 + nrow > Nq ? 0 : q0) + qoff;              // of the tile's rows
    const int pos_max = min(q0 + nrow, Nq) - 1 + qoff;
    const size_t flat0 = (size_t)bk * (p.Hq / p.Hkv * Nq);             // the group's first row in q, out, lse and counts
    // blocks the tile visits, and this workgroup's range of them
    const int nbt = causal ? pos_max / BC + 1 : (Nk + BC - 1) / BC;
    const int it0 = PHASE == 0 ? 0 : (int)((long long)nbt * cidx / C);
    const int it1 = PHASE == 0 ? nbt : (int)((long long)nbt * (cidx + 1) / C);
    auto jof = [&](int it) __attribute__((always_inline)) { return p.order == 0 ? it : nbt - 1 - it; };

    const uint8_t* Qg = static_cast<const uint8_t*>(p.q) + flat0 * KROW;
    const uint8_t* Kg = static_cast<const uint8_t*>(p.k) + (size_t)bk * Nk * KROW;
    const uint8_t* Vg = static_cast<const uint8_t*>(p.v) + (size_t)bk * Nk * D;

    // ---- K tile kt of a block: load i fills segment i / IPS, rows (i % IPS)
    // 1024 / SEG on; lane l row l / SCH of those, chunk l % SCH of the segment.
    // LDS row m of the buffer is A row m of the MFMA (key a_key(m)) ----
    const int krow = lane / SCH;
    const int k_lane = TL::a_key(krow) * KROW + 16 * (lane % SCH);
    i32x4 kr[RING][NP];
    // block at visit position it; past the range: no bytes
    auto kbuf = [&](int it) __attribute__((always_inline)) {
        const int t0 = it < it1 ? jof(it) * BC : 0;
        return row_buffer(Kg + (size_t)t0 * KROW, it < it1 ? (size_t)(Nk - t0) * KROW : 0);
    };
    auto kload = [&](__amdgpu_buffer_rsrc_t kb, int kt) __attribute__((always_inline)) {
        // (1024 / SEG rows on are 8 keys (TR = 32) or 2 GSTEP keys (TR = 16) on)
        constexpr int USTEP = (TR == 32 ? 8 : 2 * TL::GSTEP) * KROW;
#pragma unroll
        for (int i = 0; i < NP; ++i)
            kr[kt % RING][i] = __builtin_bit_cast(
                i32x4, __builtin_amdgcn_raw_buffer_load_b128(kb, k_lane + SEG * (i / IPS),
                                                             TL::TSTEP * kt * KROW + USTEP * (i % IPS), 0));
    };
    auto kissue = [&](__amdgpu_buffer_rsrc_t kb) __attribute__((always_inline)) {
#pragma unroll
        for (int kt = 0; kt < RING; ++kt)
            kload(kb, kt);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto frag8 = [](const i32x4* x) __attribute__((always_inline)) {
        if constexpr (PPS == 2)
            return i32x8{x[0][0], x[0][1], x[0][2], x[0][3], x[1][0], x[1][1], x[1][2], x[1][3]};
        else
            return i32x8{x[0][0], x[0][1], x[0][2], x[0][3], 0, 0, 0, 0};
    };
    // The wave's K buffer: row m's chunk c at chunk c ^ kswz(m), so that the 16
    // rows of a fragment read (one chunk) and the rows of a write fall in
    // distinct banks.  LDS operations of one wave run in order, so a segment
    // overwrites the one before without a wait.
    uint8_t* const kst = lds + KB_OFF + w * KB_BYTES;
    auto kswz = [](int m) __attribute__((always_inline)) { return (m / (256 / SEG)) & (SCH - 1); };
    const int k_wr = krow * SEG + 16 * ((lane % SCH) ^ kswz(krow));
    const uint8_t* const k_rd = kst + n * SEG;
    // segment i of the tiles: write it, read this lane's fragments of it
    auto kstage = [&](int i, i32x4* fr) __attribute__((always_inline)) {
        const int kt = i / NSEG, sg = i % NSEG;
        // (rows 8 on with SEG = 128 flip bit 2 of the swizzle, 16 on with SEG = 64 none)
#pragma unroll
        for (int u = 0; u < IPS; ++u)
            *reinterpret_cast<i32x4*>(kst + (SEG == 128 ? k_wr ^ (64 * u) : k_wr) + 1024 * u) = kr[kt % RING][sg * IPS + u];
#pragma unroll
        for (int q = 0; q < SPS * PPS; ++q) {
            const int chunk = PPS == 2 ? NG * 2 * (q / 2) + 2 * g + q % 2 : NG * q + g;
            fr[q] = *reinterpret_cast<const i32x4*>(k_rd + ((chunk ^ kswz(n)) << 4));
        }
    };

    uint8_t* vst = lds + (PHASE == 1 ? 0 : w * V_BYTES);
    auto vswz = [](int r) __attribute__((always_inline)) { return ((r / (256 / VROW)) & (VCPR / 2 - 1)) * 2; };
    // V of a block -> this wave's LDS stage, straight from HBM: round i writes
    // LDS bytes [1024 i, +1024); lane l fills row i V_RPI + l / VCPR at physical
    // chunk l % VCPR, which holds logical chunk (l % VCPR) ^ vswz(row).  Keys
    // past the cache end are written as 0.
    // (V_RPI is a multiple of 256 / VROW and VCPR / 2 divides V_RPI / (256 /
    // VROW), so the swizzle of row i V_RPI + l / VCPR does not depend on i: one
    // lane offset and a uniform row step)
    static_assert(V_RPI % (256 / VROW) == 0 && (V_RPI / (256 / VROW)) % (VCPR / 2) == 0,
                  "the V swizzle repeats every round");
    const int v_voff = (lane / VCPR) * D + DO * colp + 16 * ((lane % VCPR) ^ vswz(lane / VCPR));
    auto issue_v = [&](int it) __attribute__((always_inline)) {
        const int t0 = it < it1 ? jof(it) * BC : 0;
        const auto vb = row_buffer(Vg + (size_t)t0 * D, it < it1 ? (size_t)(Nk - t0) * D : 0);
#pragma unroll
        for (int i = 0; i < V_NI; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, (__attribute__((address_space(3))) void*)(vst + 1024 * i), 16,
                                                     v_voff, V_RPI * D * i, 0, 0);
    };

    // PHASE 2: the maxima of every range of the tile (C * TR <= 64 NW of them)
    float range_max = -INFINITY;
    if constexpr (PHASE == 2) {
        if (tid < C * TR)
            range_max = p.ws_max[(size_t)unit * C * TR + tid];
    }
    // Q^T fragments (B operand): the same pieces of Q[row]
    i32x4 qf[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i)
        qf[i] = row < rows ? *reinterpret_cast<const i32x4*>(Qg + (size_t)row * KROW + KSB * (i / PPS) + 16 * PPS * g + 16 * (i % PPS))
                           : i32x4{};
    // The first block's K and V are requested with them.  From here on every
    // wave issues the same loads in every round (empty ones past its range):
    // with one straight path the compiler's waits count exactly the loads that
    // are younger than the one needed, instead of draining them all.
    kissue(kbuf(it0 + w));
    if constexpr (PHASE != 1)
        issue_v(it0 + w);
    if (COUNT && tid < TR * 3)
        csh[tid / 3][tid % 3] = 0u;

    // ---- S^T = K_j Q^T over the tiles in flight; -inf for keys past the cache
    // end or past the row's position; the row maxima ----
    Acc s[KT];
    // (a tile's registers take the next tile of the ring as soon as it is used:
    // the block's, then the first ones of the wave's next block, which travel
    // during the softmax and P.V)
    auto qk = [&](int it) __attribute__((always_inline)) {
        const auto kb = kbuf(it), kb_next = kbuf(it + NW);
        i32x4 fr[2][SPS * PPS];
        constexpr int NS = KT * NSEG;
        auto stage = [&](int i) __attribute__((always_inline)) {
            kstage(i, fr[i & 1]);
            const int kt = i / NSEG;
            if (i % NSEG == NSEG - 1)
                kload(kt + RING < KT ? kb : kb_next, kt + RING < KT ? kt + RING : kt + RING - KT);
            __builtin_amdgcn_sched_barrier(0);
        };
        stage(0);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int kt = i / NSEG, sg = i % NSEG;
            if (i + 1 < NS)
                stage(i + 1);
#pragma unroll
            for (int ks = 0; ks < SPS; ++ks) {
                const int kk = sg * SPS + ks;
                const Acc acc = kk == 0 ? Acc{} : s[kt];
                if constexpr (QK8)
                    s[kt] = TL::template f8<false>(frag8(&fr[i & 1][ks * PPS]), frag8(&qf[kk * PPS]), acc, 0);
                else
                    s[kt] = TL::qk16(__builtin_bit_cast(bf16x8, fr[i & 1][ks]), __builtin_bit_cast(bf16x8, qf[kk]), acc);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // last valid key of the row in the block at t0 (its own offset), -1: none
    auto limit = [&](bool on, int t0) __attribute__((always_inline)) {
        return on ? (causal ? min(pos, Nk - 1) : Nk - 1) - t0 : -1;
    };
    auto mask = [&](bool on, int t0) __attribute__((always_inline)) {
        if (!on || (causal && t0 + BC - 1 > pos_min) || t0 + BC > Nk) {
            const int lim = limit(on, t0) - TL::GSTEP * g;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < REGS; ++r) {
                    const uint32_t m = (uint32_t)((lim - (TL::TSTEP * kt + r)) >> 31);
                    s[kt][r] = __uint_as_float((__float_as_uint(s[kt][r]) & ~m) | (0xFF800000u & m));
                }
        }
    };
    auto over_groups_max = [](float x) __attribute__((always_inline)) {
        x = halves_max(x);
        if constexpr (NG == 4)
            x = fmax_f(x, __shfl_xor(x, 16, 64));
        return x;
    };
    auto over_groups_sum = [](float x) __attribute__((always_inline)) {
        if constexpr (NG == 4)
            x += __shfl_xor(x, 16, 64);
        return halves_sum(x);
    };
    auto row_max = [&]() __attribute__((always_inline)) {
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < REGS; ++r)
                mx = fmax_f(mx, s[kt][r]);
        return mx;
    };

    const int rounds = (it1 - it0 + NW - 1) / NW;
    if constexpr (PHASE == 1) {
        float m1 = -INFINITY;
        for (int rd = 0; rd < rounds; ++rd) {
            const int it = it0 + rd * NW + w;
            qk(it);
            mask(it < it1, jof(it) * BC);
            m1 = fmax_f(m1, row_max());
        }
        m1 = over_groups_max(m1);
        if (g == 0)
            tab[0][w][n] = m1;
        lds_barrier();
        if (tid < TR) {
            float m = tab[0][0][tid];
#pragma unroll
            for (int v = 1; v < NW; ++v)
                m = fmax_f(m, tab[0][v][tid]);
            p.ws_max[((size_t)unit * C + cidx) * TR + tid] = m;
        }
        return;
    }

    // the running maximum before this workgroup's range, and the final one
    float carry = -INFINITY, m_final = -INFINITY;
    if constexpr (PHASE == 2) {
        rmax[tid] = range_max;
        lds_barrier();
        for (int cc = 0; cc < C; ++cc) {
            const float t = rmax[cc * TR + n];
            if (cc < cidx)
                carry = fmax_f(carry, t);
            m_final = fmax_f(m_final, t);
        }
    }

    const float c = p.c;
    const float S = p.S;
    float m_run = -INFINITY;            // the running maximum after this wave's last block
    float mc_run = -INFINITY;
    float ell = 0.f;
    Acc o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        o[dt] = Acc{};
    uint32_t cnt0 = 0, cnt1 = 0, cnt2 = 0;

    const int j16 = lane & 15;
    // V^T operand: TR = 32: rows 16 g + {0, 8, 32, 40} + 64 js, chunk 2 dt +
    // (n >> 4); TR = 16: rows (BC / 4) g + 8 i, chunk dt; row j16 >> 1, half
    // j16 & 1 of the chunk in the transposed read of a 16-lane group
    const uint32_t v_lane = (uint32_t)(((j16 >> 1) + TL::GSTEP * g) * VROW + (((TR == 32 ? n >> 4 : 0) ^ vswz(j16 >> 1)) << 4) +
                                       8 * (j16 & 1));

    for (int rd = 0; rd < rounds; ++rd) {
        const int it = it0 + rd * NW + w;
        const bool on = it < it1;
        const int j = jof(it);
        const int t0 = j * BC;
        qk(it);
        mask(on, t0);
        const float mx = over_groups_max(row_max());
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
        // (a wave past the range goes on with every key masked: P = 0)
        const float m_new = fmax_f(m_prev, mx);
        const float mc_new = m_new * c;
        // before the row's first valid key nothing has accumulated: alpha is
        // irrelevant and P must be 0 (x = -inf), not NaN
        const bool none = mc_new == -INFINITY;
        const float alpha = none ? 1.f : __builtin_amdgcn_exp2f(mc_run - mc_new);
        const float nmc = none ? 0.f : -mc_new;
        float cvt_scale = p.inv_S;
        int pv_sb = 127;
        if constexpr (SCALE == kScaleDynamic) {
            const float xmax = __builtin_fmaf(mx, c, nmc);
            const float f = __builtin_fminf(__builtin_fmaxf(__builtin_floorf(-xmax), 0.f),
                                            (float)(126 - p.k0));
            const int kj = p.k0 + (int)f;
            cvt_scale = __uint_as_float((uint32_t)(127 - kj) << 23);
            pv_sb = 127 + p.k0 - kj;
        }
        float lsum = 0.f;
        uint32_t pk[8 * PVS] = {};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            float ps[REGS];
#pragma unroll
            for (int r = 0; r < REGS; ++r)
                ps[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r], c, nmc));
#pragma unroll
            for (int r = 0; r < REGS; ++r)
                lsum += ps[r];
#pragma unroll
            for (int r4 = 0; r4 < REGS / 4; ++r4) {
                const float p0 = ps[4 * r4 + 0], p1 = ps[4 * r4 + 1];
                const float p2 = ps[4 * r4 + 2], p3 = ps[4 * r4 + 3];
                uint32_t word;
                if constexpr (SCALE != kScaleAny) {
                    s16x2 lo = {};
                    lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(lo, p0, p1, cvt_scale, false);
                    lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(lo, p2, p3, cvt_scale, true);
                    word = __builtin_bit_cast(uint32_t, lo);
                } else {
                    int wv = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_fminf(p0 * S, 448.f),
                                                            __builtin_fminf(p1 * S, 448.f), 0, false);
                    wv = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_fminf(p2 * S, 448.f),
                                                        __builtin_fminf(p3 * S, 448.f), wv, true);
                    word = (uint32_t)wv;
                }
                pk[kt * (REGS / 4) + r4] = word;
                if (COUNT || TR == 32)
                    __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (COUNT) {
            // byte i of word (kt, r4) holds the block's key k0 + i; it is valid iff
            // k0 + i <= lim, and a sink key iff k0 + i < ns (invalid and
            // other-category bytes are forced non-zero)
            const int lim = limit(on && row < rows, t0);
            const int ns = j == 0 ? p.n_sink : 0;
            auto low_bytes = [](int x) __attribute__((always_inline)) {
                return (uint32_t)((1ull << (8 * min(max(x, 0), 4))) - 1);
            };
            uint32_t z0 = 0, zn = 0;
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                const int k0 = TL::TSTEP * (i / (REGS / 4)) + TL::GSTEP * g + 4 * (i % (REGS / 4));
                const uint32_t valid = low_bytes(lim - k0 + 1);
                if (j == 0) {
                    const uint32_t sink = low_bytes(ns - k0);
                    z0 += zero_codes(pk[i] | ~(valid & sink));
                    zn += zero_codes(pk[i] | ~(valid & ~sink));
                } else {
                    zn += zero_codes(pk[i] | ~valid);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            cnt0 += z0;
            cnt1 += j == 0 ? zn : 0u;
            cnt2 += j == 0 ? 0u : zn;
        }
        ell = alpha * ell + lsum;
        // (alpha is exactly 1 in every lane while no row's maximum moves)
        if (__ballot(alpha != 1.0f) != 0) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < REGS; ++r)
                    o[dt][r] *= alpha;
        }
        m_run = m_new;
        mc_run = mc_new;

        // ---- O^T += V_j^T P8^T ----
        // (this block's V is older than the next block's K: wait for all but those)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(RING * NP) : "memory");
        // (the V^T operands are read one MFMA ahead; the fences keep the compiler
        // from reading them all at once, which spills)
        constexpr int NM = PVS * DT;
        auto vread = [&](int i) __attribute__((always_inline)) {
            const int js = i / DT, dt = i % DT;
            i32x8 av = {};
#pragma unroll
            for (int u = 0; u < (PW < 8 ? PW / 2 : 4); ++u) {
                const int vrow = TR == 32 ? 64 * js + 32 * (u / 2) + 8 * (u % 2) : 8 * u;
                const i32x2 t = read_tr8(vst + (v_lane ^ (uint32_t)(dt << (TR == 32 ? 5 : 4))) + vrow * VROW);
                av[2 * u] = t[0];
                av[2 * u + 1] = t[1];
            }
            return av;
        };
        i32x8 av[2];
        av[0] = vread(0);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int js = i / DT, dt = i % DT;
            if (i + 1 < NM)
                av[(i + 1) & 1] = vread(i + 1);
            i32x8 bop;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                bop[q] = (int)pk[8 * js + q];
            __builtin_amdgcn_sched_barrier(0);
            o[dt] = TL::template f8<SCALE == kScaleDynamic>(av[i & 1], bop, o[dt], pv_sb);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the next block's V: its stage is free once the last read of this
        // one has returned
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue_v(it + NW);
    }
    if constexpr (PHASE == 0)
        m_final = carry;

    // ---- merge: bring each wave's (O, l) to the rows' final maximum and sum ----
    const float mc_final = m_final * c;
    const float beta = mc_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc_run - mc_final);
    const float ell_w = over_groups_sum(ell) * beta;
    if (COUNT) {
        auto add = [](uint32_t x) __attribute__((always_inline)) {
            if constexpr (NG == 4)
                x += (uint32_t)__shfl_xor((int)x, 16, 64);
            return x + other_half_u32(x);
        };
        cnt0 = add(cnt0);
        cnt1 = add(cnt1);
        cnt2 = add(cnt2);
    }
    // the V stages become the merge buffer (the last, empty V loads write zeros:
    // they have to have landed)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    float* const mw = reinterpret_cast<float*>(lds) + (w * TR + n) * MS;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < REGS / 4; ++r4) {
            f32x4 v4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v4[i] = o[dt][4 * r4 + i] * beta;
            *reinterpret_cast<f32x4*>(mw + TR * dt + TL::d_row(4 * r4, g)) = v4;
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
    const float* mb = reinterpret_cast<const float*>(lds);
    float* const part = PHASE == 2 ? p.ws_part + ((size_t)unit * C + cidx) * (TR * D + TR) : nullptr;
    for (int e = tid; e < TR * DO / 4; e += 64 * NW) {
        const int rr = e / (DO / 4), piece = e % (DO / 4);
        if (row0 + rr >= rows)
            continue;
        f32x4 acc = *reinterpret_cast<const f32x4*>(mb + rr * MS + 4 * piece);
        float l = lsh[0][rr];
#pragma unroll
        for (int v = 1; v < NW; ++v) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(mb + (v * TR + rr) * MS + 4 * piece);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i] += t[i];
            l += lsh[v][rr];
        }
        if constexpr (PHASE == 2) {
            // this workgroup's sum (at the tile's final maximum)
            *reinterpret_cast<f32x4*>(part + 4 * e) = acc;
        } else if (p.out) {
            const float inv = p.v_descale / (S * l);
            f32x4 v4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v4[i] = acc[i] * inv;
            *reinterpret_cast<f32x4*>(p.out + (flat0 + row0 + rr) * D + DO * colp + 4 * piece) = v4;
        }
    }
    if (colp == 0 && tid < TR && row < rows) {      // lane tid of wave 0 holds row tid: m_final is that row's maximum
        const size_t flat = flat0 + row;
        float l = lsh[0][tid];
#pragma unroll
        for (int v = 1; v < NW; ++v)
            l += lsh[v][tid];
        if constexpr (PHASE == 2)
            part[TR * D + tid] = l;
        else if (p.lse)
            p.lse[flat] = (mc_final + __builtin_log2f(l)) * 0.6931471805599453f;
        if (COUNT) {
            if constexpr (PHASE == 2) {
                // the host clears the counts before a split launch
                atomicAdd(p.counts + 3 * flat + 0, csh[tid][0]);
                atomicAdd(p.counts + 3 * flat + 1, csh[tid][1]);
                atomicAdd(p.counts + 3 * flat + 2, csh[tid][2]);
            } else {
                p.counts[3 * flat + 0] = csh[tid][0];
                p.counts[3 * flat + 1] = csh[tid][1];
                p.counts[3 * flat + 2] = csh[tid][2];
            }
        }
    }
}

namespace {

template <int D, int BC, bool COUNT, bool QK8, int TR>
hipError_t kv_launch(const Params& p, int scale, int phase, int cols, int waves, hipStream_t s)
{
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(p.per_xcd * kNumXcd), dim3(64 * waves), 0, s, p);
        return hipGetLastError();
    };
    auto by_scale = [&](auto ph, auto ds, auto nw) {
        constexpr int PH = decltype(ph)::value, DS = decltype(ds)::value, NW = decltype(nw)::value;
        return scale == kScaleDynamic ? go(kv_kernel<D, BC, COUNT, kScaleDynamic, QK8, TR, PH, DS, NW>)
               : scale == kScalePow2  ? go(kv_kernel<D, BC, COUNT, kScalePow2, QK8, TR, PH, DS, NW>)
                                      : go(kv_kernel<D, BC, COUNT, kScaleAny, QK8, TR, PH, DS, NW>);
    };
    using std::integral_constant;
    constexpr integral_constant<int, 0> unsplit{};
    constexpr integral_constant<int, 1> one{};
    constexpr integral_constant<int, 2> two{};
    constexpr integral_constant<int, 4> w4{};
    constexpr integral_constant<int, 8> w8{};
    if (phase == 1)   // only maxima: one instantiation, whatever the scale and diagnostics
        return go(kv_kernel<D, BC, false, kScaleAny, QK8, TR, 1, 1, 8>);
    if (phase == 2)
        return by_scale(two, one, w8);
    if (cols == 2) {
        if constexpr (TR == 16 && kv_cols_built(D, BC, QK8, 8)) {
            if (waves == 8)
                return by_scale(unsplit, two, w8);
        }
        if constexpr (TR == 16 && kv_cols_built(D, BC, QK8, 4)) {
            if (waves == 4)
                return by_scale(unsplit, two, w4);
        }
        return hipErrorInvalidValue;   // (no plan asks for it)
    }
    return waves == 4 ? by_scale(unsplit, one, w4) : by_scale(unsplit, one, w8);
}

}  // namespace

template <bool QK8, int TR>
hipError_t launch_kv_t(const Params& p, int d, int block_kv, bool count, int scale, int phase, int cols, int waves,
                       hipStream_t s)
{
    auto pick = [&](auto dc, auto bc) {
        constexpr int D = decltype(dc)::value, BC = decltype(bc)::value;
        return count ? kv_launch<D, BC, true, QK8, TR>(p, scale, phase, cols, waves, s)
                     : kv_launch<D, BC, false, QK8, TR>(p, scale, phase, cols, waves, s);
    };
    using std::integral_constant;
    if (d == 64)
        return block_kv == 64 ? pick(integral_constant<int, 64>{}, integral_constant<int, 64>{})
                              : pick(integral_constant<int, 64>{}, integral_constant<int, 128>{});
    return block_kv == 64 ? pick(integral_constant<int, 128>{}, integral_constant<int, 64>{})
                          : pick(integral_constant<int, 128>{}, integral_constant<int, 128>{});
}

}  // namespace attn
