// KV-cache kernel, bf16 Q/K, 32-row tiles.
#include "attn_prefill_kernel.hpp"

namespace attn {
template hipError_t launch_kv_t<false, 32>(const Params&, int, int, bool, int, int, int, int, hipStream_t);
}  // namespace attn
