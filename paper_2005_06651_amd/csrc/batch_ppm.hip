// batch_ppm.hip -- fused stage kernels of batched blocks with PPM reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_batch<Tile<18, 14>, 2>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<14, 18>, 2>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<16, 16>, 2>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<18, 10>, 2>(int, const BatchArgs&, int, hipStream_t, bool);
}  // namespace athmhd
