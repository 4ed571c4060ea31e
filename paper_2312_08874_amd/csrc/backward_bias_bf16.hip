// The recomputing backward's kernels for problems with an agent bias, element type bf16.
#include "backward_fused.inc"

namespace aa {
template hipError_t launch_token<ElemBF16, true>(int, int, int, const TokenArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_agent<ElemBF16, true>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_both<ElemBF16, true>(int, int, const AgentArgs&, dim3, size_t, hipStream_t);
}  // namespace aa
