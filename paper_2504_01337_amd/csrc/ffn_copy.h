// Asynchronous global -> LDS copies of the bf16 expert-FFN kernels, and the waits and barriers that go with them.
#pragma once
#include "c2r_internal.h"

namespace c2r {

// 16 bytes per lane, global -> LDS, without passing through registers.  `lds` is the
// wave-uniform start of the 1024-byte run; lane l's data lands at lds + 16*l.
// Written as inline assembly on purpose: when the compiler sees the copy as an LDS write
// it guards later LDS reads with vmcnt(0) whenever its alias bookkeeping loses track
// (it does across unrolled rings), which serialises the pipeline.  Hidden
// from it, the only waits on copies are the ones the kernels state (wait_copies_but).
// The source is a wave-uniform base (scalar registers) plus a 32-bit byte offset per lane:
// no 64-bit address arithmetic per copy, and half the address bits to send.
__device__ __forceinline__ void copy16_to_lds(const unsigned char *base, uint32_t off, unsigned char *lds) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    asm volatile(
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(off), "s"(base), "s"(lds_addr)
        : "memory", "m0");
#endif
}

// A pointer the compiler may keep in scalar registers (the value is the same in every lane).
__device__ __forceinline__ const unsigned char *uniform_ptr(const unsigned char *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const unsigned char *>(((uint64_t)hi << 32) | lo);
}

// Wait until at most N of this wave's copies are still in flight (they complete in order);
// the other counters are left alone.
template <int N>
__device__ __forceinline__ void wait_copies_but() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
#endif
}

// vmcnt(0) and lgkmcnt(0): this wave's copies have landed and its LDS reads have returned.
__device__ __forceinline__ void wait_copies_and_lds() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0070);
#endif
}

// lgkmcnt(0) alone: this wave's LDS reads have returned and its LDS writes are done; whatever
// it has in flight to or from memory (the epilogue's stores) stays in flight.
__device__ __forceinline__ void wait_lds_only() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0xC07F);
#endif
}

// Same, and this wave's LDS reads have returned (lgkmcnt(0)).
template <int N>
__device__ __forceinline__ void wait_copies_but_and_lds() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
#endif
}

// Bare workgroup barrier.  __syncthreads() (and any workgroup fence) also drains every
// outstanding copy (vmcnt(0)), which would serialise the slices in flight; here the
// caller states exactly which copies must have landed (wait_copies_but) and the
// scheduling fences keep the compiler from moving LDS reads across the barrier.
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// What this wave wrote to LDS is there, then the workgroup's barrier; loads in flight into registers stay in flight (a
// __syncthreads() would wait for them).  The clobber keeps the compiler from moving or forwarding LDS accesses across.
__device__ __forceinline__ void lds_hand_over() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

}  // namespace c2r
