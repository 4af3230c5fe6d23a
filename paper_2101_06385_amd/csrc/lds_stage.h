// LDS stages filled by direct loads (global_load_lds issued from inline asm), shared by the
// kernels that pipeline them.
#pragma once

#include <hip/hip_runtime.h>

namespace sp2 {
namespace {

// The barrier between the reads of a stage and the direct loads that refill it: every LDS read of
// this wave has returned, so behind the barrier other waves' loads may take its place.
// __syncthreads does not promise that: the compiler does not see the direct loads as LDS
// writes and may leave reads in flight across it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
}  // namespace sp2
