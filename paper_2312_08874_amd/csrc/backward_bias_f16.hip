// The recomputing backward's kernels for problems with an agent bias, element type f16.
#include "backward_fused.inc"

namespace aa {
template hipError_t launch_token_bias<ElemF16>(int, int, const TokenArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_agent_bias<ElemF16>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
}  // namespace aa
