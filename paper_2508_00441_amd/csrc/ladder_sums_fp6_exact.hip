#include "ladder_sums.hpp"

namespace ozaki {

template hipError_t launch_ladder_kernel<FMT_FP6, ACC_EXACT>(const LadderArgs&, int, int, unsigned, hipStream_t);

}  // namespace ozaki
