// The recomputing kernels for fp32 elements: the backward pass, and the forward pass of problems that the one-launch
// fp32 kernel does not serve.
#include "backward_fused.inc"

namespace aa {
template hipError_t launch_token<ElemF32, false>(int, int, int, const TokenArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_token<ElemF32, true>(int, int, int, const TokenArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_agent<ElemF32, false>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_agent<ElemF32, true>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_both<ElemF32, false>(int, int, const AgentArgs&, dim3, size_t, hipStream_t);
template hipError_t launch_both<ElemF32, true>(int, int, const AgentArgs&, dim3, size_t, hipStream_t);
}  // namespace aa
