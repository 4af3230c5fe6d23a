// One-workgroup-per-tile split squaring kernels (single and grouped), FP16 planes.
#include "k_square_sk.h"

namespace sp2 {
template hipError_t launch_dp_t<_Float16>(int tile, int variant, const SquareArgs& a, const SquareArgs* descs,
                                       const TileRef* map, int per, hipStream_t s);
}  // namespace sp2
