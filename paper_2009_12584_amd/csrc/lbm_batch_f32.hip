// Batched step kernels with FP32 deviation storage (lbm_batch_kernels.hpp).
#include "lbm_batch_kernels.hpp"

namespace mclbm {
void launch_batch_f32(const BatchLaunch &B, hipStream_t s, int lp, long long L, bool diag) {
    launch_batch_storage<float>(B, s, lp, L, diag);
}
void launch_batch_sweep_f32(const BatchLaunch &B, hipStream_t s, int lp, long long L) {
    launch_batch_sweep<float>(B, s, lp, L);
}
}  // namespace mclbm
