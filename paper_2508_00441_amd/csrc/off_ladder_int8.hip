#include "off_ladder.hpp"

namespace ozaki {

template hipError_t launch_off_ladder_format<FMT_INT8>(const OffLadderArgs&, int, bool, unsigned, hipStream_t);

}  // namespace ozaki
