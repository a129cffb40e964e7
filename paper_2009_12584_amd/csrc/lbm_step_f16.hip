// Step kernels of one simulation with FP16 deviation storage (lbm_step_kernels.hpp).
#include "lbm_step_kernels.hpp"

namespace mclbm {
void launch_step_f16(const Launch &L, dim3 g, hipStream_t s, const Inst &I, int parity, const Fields &fo,
                     double *partials) {
    launch_storage<__half>(L, g, s, I, parity, fo, partials);
}
void launch_sweep_f16(const Launch &L, hipStream_t s, const Inst &I, const SweepPlan &W, int parity) {
    launch_sweep_storage<__half>(L, s, I, W, parity);
}
}  // namespace mclbm
