// The 256 x 256 slice-pair GEMM kernels whose runs may pass the window's worst case (RunCheck in layout.hpp).
#include "pair_gemm_body.hpp"

namespace ozaki {

namespace {

template <int FMT>
__global__ void __launch_bounds__(256) pair_gemm_measured_kernel(const GemmArgs a) { pair_gemm_body<FMT, true>(a); }

}  // namespace

hipError_t launch_pair_gemm_measured(const GemmArgs& a, int fmt, unsigned blocks, hipStream_t st) {
    const dim3 grid(blocks), block(256);
    if (fmt == FMT_FP16) hipLaunchKernelGGL((pair_gemm_measured_kernel<FMT_FP16>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6) hipLaunchKernelGGL((pair_gemm_measured_kernel<FMT_FP6>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((pair_gemm_measured_kernel<FMT_FP6_E3M2>), grid, block, 0, st, a);
    else if (fmt == FMT_FP8) hipLaunchKernelGGL((pair_gemm_measured_kernel<FMT_FP8>), grid, block, 0, st, a);
    else return hipErrorInvalidValue;             // INT8: the window holds every anti-diagonal anyway
    return hipGetLastError();
}

}  // namespace ozaki
