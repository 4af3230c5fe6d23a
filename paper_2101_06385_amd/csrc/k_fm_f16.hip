// Fragment-major split squaring kernels, FP16 planes.
#include "k_square_fm.h"

namespace sp2 {
template hipError_t launch_fm_t<_Float16>(int variant, const FmArgs& a, hipStream_t s);
}  // namespace sp2
