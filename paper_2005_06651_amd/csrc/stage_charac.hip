// stage_charac.hip -- fused stage kernels of uniform blocks with PLM on
// characteristic variables.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_charac<TileU>(int, const UniformArgs&, hipStream_t);
template hipError_t launch_charac<TileS>(int, const UniformArgs&, hipStream_t);
}  // namespace athmhd
