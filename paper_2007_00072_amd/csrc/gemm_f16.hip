// The contraction kernels of gemm_kernels.hpp for fp16 storage (one
// translation unit per storage type, so that they compile side by side).
#include "gemm_kernels.hpp"

namespace dm {

void launch_tiles_f16(const GemmArgs& g, hipStream_t st) { launch_t<half_t>(g, st); }
void launch_reduce_f16(const GemmArgs& g, hipStream_t st) { launch_reduce<half_t>(g, st); }
void launch_pair_f16(const GemmArgs& g0, const GemmArgs& g1, hipStream_t st) {
    launch_lean_pair<half_t, 128, 128, 2, 4, 64, 4>(g0, g1, st);
}

}  // namespace dm
