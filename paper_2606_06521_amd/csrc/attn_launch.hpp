// Host-side launchers of the two kernel families (defined next to their
// kernels) and the tile geometry the dispatcher needs to size the grid.
#pragma once

#include "attn_common.hpp"
#include "attn_plan.hpp"

namespace attn {

// sets its own tile geometry and grid in p
hipError_t launch_faithful(const Params& p, int d, int block_kv, bool causal, bool count,
                           bool cast, int scale, int n_cu, hipStream_t stream);

// The fast kernel (persistent): QK8 selects E4M3 Q and K (S^T on the FP8
// MFMA), PAIR the 128-row schedule (two waves per 32-row group, alternate
// blocks).  grid: a multiple of 8 workgroups, at most one per CU; scale: kScale*.
// Each (QK8, PAIR) pair is instantiated in its own translation unit.
template <bool QK8, bool PAIR>
hipError_t launch_fast_t(const Params& p, int grid, int d, int block_kv, bool causal, bool count, int scale,
                         hipStream_t stream);
extern template hipError_t launch_fast_t<false, false>(const Params&, int, int, int, bool, bool, int, hipStream_t);
extern template hipError_t launch_fast_t<false, true>(const Params&, int, int, int, bool, bool, int, hipStream_t);
extern template hipError_t launch_fast_t<true, false>(const Params&, int, int, int, bool, bool, int, hipStream_t);
extern template hipError_t launch_fast_t<true, true>(const Params&, int, int, int, bool, bool, int, hipStream_t);
// The KV-cache kernel by its plan: one workgroup per (batch, KV head, tile of the
// group's query rows), or several (over the keys: three launches on the stream and
// a workspace of plan.bytes); sets its own grid, nsplit and workspace fields of p
hipError_t launch_prefill(const Params& p, const KvPlan& plan, int d, int block_kv, bool causal, bool count,
                          int scale, bool qk8, void* ws, hipStream_t stream);
// One launch of the KV-cache kernel: phase 0 (unsplit), 1 (range maxima) or 2
// (the visit per range); cols: workgroups per tile that share its columns (phase
// 0, TR = 16); waves per workgroup: 8, or 4 (phase 0); QK8 selects E4M3 Q and K, TR the tile height.  Each
// pair is instantiated in its own translation unit.
template <bool QK8, int TR>
hipError_t launch_kv_t(const Params& p, int d, int block_kv, bool count, int scale, int phase, int cols,
                       int waves, hipStream_t s);
extern template hipError_t launch_kv_t<false, 16>(const Params&, int, int, bool, int, int, int, int, hipStream_t);
extern template hipError_t launch_kv_t<true, 16>(const Params&, int, int, bool, int, int, int, int, hipStream_t);
extern template hipError_t launch_kv_t<false, 32>(const Params&, int, int, bool, int, int, int, int, hipStream_t);
extern template hipError_t launch_kv_t<true, 32>(const Params&, int, int, bool, int, int, int, int, hipStream_t);

}  // namespace attn
