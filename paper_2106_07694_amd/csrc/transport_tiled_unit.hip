// transport_tiled_unit.hip -- one unit of the tiled RK3 stage kernels.  Built
// once per element type (LBW_T), dimension (LBW_D) and settling form (LBW_VSS:
// 1 when the settling speed depends on S), so the eight units compile in
// parallel.
#include "transport_tiled.h"

namespace lbw {
template hipError_t tiled_unit<LBW_T, LBW_D, LBW_VSS != 0>(const RunDev &, const ClassSet &,
                                                           const TileShape &, int, hipStream_t,
                                                           const BatchArgs *);
}  // namespace lbw
