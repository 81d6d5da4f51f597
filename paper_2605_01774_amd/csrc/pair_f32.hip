// Two-step launcher for the F32 storage form.
#include "pair_kernel.h"

namespace elbm {

hipError_t launch_step_pair_f32(const elbm_lattice* h, const void* src, void* dst, const StepPair& p, bool* done) {
    return step_pair<float>(h, src, dst, p, done);
}

}  // namespace elbm
