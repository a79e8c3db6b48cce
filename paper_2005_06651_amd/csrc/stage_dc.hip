// stage_dc.hip -- fused stage kernels of uniform blocks with DC reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_uniform<0, TileU>(int, const UniformArgs&, hipStream_t);
template hipError_t launch_uniform<0, TileS>(int, const UniformArgs&, hipStream_t);
}  // namespace athmhd
