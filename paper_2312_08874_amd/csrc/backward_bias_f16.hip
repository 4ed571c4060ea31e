// The recomputing backward's kernels for problems with an agent bias, element type f16.
#include "backward_fused.inc"

namespace aa {
template hipError_t launch_token<ElemF16, true>(int, int, int, const TokenArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_agent<ElemF16, true>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_both<ElemF16, true>(int, int, const AgentArgs&, dim3, size_t, hipStream_t);
}  // namespace aa
