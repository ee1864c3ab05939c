// LDS-staged right-hand side and fused stage: FP32 algebra, central advection.
#include "ccz4_stage_lds.hpp"

namespace ccz4 {
template hipError_t launch_rhs_lds<float, 0>(const RhsLaunch &, hipStream_t);
template hipError_t launch_stage_lds<float, 0>(const StageLaunch &, hipStream_t);
}  // namespace ccz4
