// stage_plm.hip -- fused stage kernels of uniform blocks with PLM reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_uniform<1, TileU>(int, const UniformArgs&, hipStream_t);
template hipError_t launch_uniform<1, TileS>(int, const UniformArgs&, hipStream_t);
}  // namespace athmhd
