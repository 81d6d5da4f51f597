// One instantiation of the one-node-per-thread kernel whose registers leave room for four wavefronts
// per SIMD and no more: D3Q27, plain BF16, velocity per node.
#include "step_kernels.h"

template __global__ void elbm::k_step<elbm::bf16s, 2, false, false, false, false>(const elbm::StepArgs<float>);
