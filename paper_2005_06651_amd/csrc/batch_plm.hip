// batch_plm.hip -- fused stage kernels of batched blocks with PLM reconstruction.
#include "stage_tile.hpp"

namespace athmhd {
template hipError_t launch_batch<Tile<18, 14>, 1>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<14, 18>, 1>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<16, 16>, 1>(int, const BatchArgs&, int, hipStream_t, bool);
template hipError_t launch_batch<Tile<18, 10>, 1>(int, const BatchArgs&, int, hipStream_t, bool);
}  // namespace athmhd
