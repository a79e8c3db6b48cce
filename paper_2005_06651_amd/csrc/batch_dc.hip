// batch_dc.hip -- fused stage kernels of batched blocks with DC reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_batch<Tile<18, 14>, 0>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<14, 18>, 0>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<16, 16>, 0>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<18, 10>, 0>(int, const BatchArgs&, int, hipStream_t, bool);
}  // namespace athmhd
