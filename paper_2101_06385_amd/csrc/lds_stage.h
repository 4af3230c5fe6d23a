// LDS stages filled by direct loads (global_load_lds issued from inline asm), shared by the
// kernels that pipeline them.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sp2 {
namespace {

typedef __attribute__((address_space(3))) unsigned char lds_byte;
__device__ __forceinline__ unsigned lds_addr(const unsigned char* p) {
    return (unsigned)(uintptr_t)(const lds_byte*)p;
}

// One 16-byte-per-lane direct load from global memory into LDS (global_load_lds_dwordx4: M0 holds
// the wave-uniform LDS base, lane L's 16 bytes land at base + 16 L), from a wave-uniform base
// address in SGPRs and a 32-bit per-lane byte offset: half the address data of the 64-bit form, and
// no per-load vector address arithmetic.  Issued from inline asm so that the compiler does not treat
// it as an LDS store it must wait for before every later LDS read: completion is tracked explicitly
// with wait_vm and a barrier before a stage is read.
__device__ __forceinline__ void dma16s(unsigned voff, const void* sbase, unsigned lds_base) {
    asm volatile(
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(voff), "s"(sbase), "s"(lds_base)
        : "memory", "m0");
}

// Waits until at most n vector-memory instructions of this wave are outstanding, n <= MAX.  s_waitcnt
// needs an immediate: n is rounded down to one of these (waiting for more than asked is always safe).
template <int MAX>
__device__ __forceinline__ void wait_vm(int n) {
    static_assert(MAX <= 48, "the largest immediate below");
#define SP2_VMCNT(k)                                             \
    if (MAX >= k && n >= k) {                                    \
        asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory");    \
        return;                                                  \
    }
    SP2_VMCNT(48) SP2_VMCNT(40) SP2_VMCNT(32) SP2_VMCNT(28) SP2_VMCNT(24) SP2_VMCNT(20) SP2_VMCNT(18) SP2_VMCNT(16)
    SP2_VMCNT(14) SP2_VMCNT(12) SP2_VMCNT(10) SP2_VMCNT(8) SP2_VMCNT(6) SP2_VMCNT(4) SP2_VMCNT(2)
#undef SP2_VMCNT
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The barrier between the reads of a stage and the direct loads that refill it: every LDS read of
// this wave has returned, so behind the barrier other waves' loads may take its place.
// __syncthreads does not promise that: the compiler does not see the direct loads as LDS
// writes and may leave reads in flight across it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
}  // namespace sp2
