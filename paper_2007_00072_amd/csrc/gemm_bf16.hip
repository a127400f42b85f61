// The contraction kernels of gemm_kernels.hpp for bf16 storage (one
// translation unit per storage type, so that they compile side by side).
#include "gemm_kernels.hpp"

namespace dm {

void launch_tiles_bf16(const GemmArgs& g, hipStream_t st) { launch_t<bf16_t>(g, st); }
void launch_reduce_bf16(const GemmArgs& g, hipStream_t st) { launch_reduce<bf16_t>(g, st); }
void launch_pair_bf16(const GemmArgs& g0, const GemmArgs& g1, hipStream_t st) {
    launch_lean_pair<bf16_t, 128, 128, 2, 4, 64, 4>(g0, g1, st);
}

}  // namespace dm
