// Two-step launcher for the F32 storage form.
#include "pair_kernel.h"

namespace elbm {

bool plan_step_pair_f32(const elbm_lattice* h, PairPlan* plan) { return plan_pair<float>(h, plan); }
hipError_t launch_step_pair_f32(const elbm_lattice* h, const void* src, void* dst, const StepPair& p,
                                const PairPlan& plan) {
    return step_pair<float>(h, src, dst, p, plan);
}

}  // namespace elbm
