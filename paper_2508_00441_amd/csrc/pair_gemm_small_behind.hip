// The slice-pair GEMMs in 128 x 128 blocks behind launch_ladder_sums.
#include "pair_gemm_small.hpp"

namespace ozaki {

hipError_t launch_pair_gemm_small_behind(const SmallGemmArgs& a, int fmt, const dim3& grid, hipStream_t st) {
    return launch_small_kernel<true>(a, fmt, grid, st);
}

}  // namespace ozaki
