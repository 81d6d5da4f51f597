// Two-step launcher for the F64 storage form.
#include "pair_kernel.h"

namespace elbm {

hipError_t launch_step_pair_f64(const elbm_lattice* h, const void* src, void* dst, const StepPair& p, bool* done) {
    return step_pair<double>(h, src, dst, p, done);
}

}  // namespace elbm
