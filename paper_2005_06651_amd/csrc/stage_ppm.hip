// stage_ppm.hip -- fused stage kernels of uniform blocks with PPM reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_uniform<2, TileU>(int, const UniformArgs&, hipStream_t);
template hipError_t launch_uniform<2, TileS>(int, const UniformArgs&, hipStream_t);
}  // namespace athmhd
