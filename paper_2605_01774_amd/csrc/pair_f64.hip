// Two-step launcher for the F64 storage form.
#include "pair_kernel.h"

namespace elbm {

bool plan_step_pair_f64(const elbm_lattice* h, PairPlan* plan) { return plan_pair<double>(h, plan); }
hipError_t launch_step_pair_f64(const elbm_lattice* h, const void* src, void* dst, const StepPair& p,
                                const PairPlan& plan) {
    return step_pair<double>(h, src, dst, p, plan);
}

}  // namespace elbm
