// LDS-staged right-hand side and fused stage: FP64 algebra, lopsided advection.
#include "ccz4_stage_lds.hpp"

namespace ccz4 {
template hipError_t launch_rhs_lds<double, 1>(const RhsLaunch &, hipStream_t);
template hipError_t launch_stage_lds<double, 1>(const StageLaunch &, hipStream_t);
}  // namespace ccz4
