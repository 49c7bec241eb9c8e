#include "ladder_sums.hpp"

namespace ozaki {

template hipError_t launch_ladder_kernel<FMT_INT8, ACC_EMU>(const LadderArgs&, int, int, unsigned, hipStream_t);

}  // namespace ozaki
