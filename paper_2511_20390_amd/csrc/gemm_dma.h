// Global memory -> LDS loads without registers in between, for the GEMM kernels whose K loop is fed by them
// (gemm_pipe.hip).  Device code.
#pragma once

#include "gemm_tile.h"

namespace freemi {

namespace {

// One block of 1 KB: lane i's 16 bytes at rsrc[voff + soff] land at LDS address lds_addr + 16 i (rows past the end of the
// matrix read as zero).  Inline assembly, because the compiler lets every LDS read wait for all such loads of the builtin
// form (it cannot tell the stages apart); wait_vm counts them by hand.  The compiler's own counts stay right: it knows of
// fewer loads in flight than there are and so waits for more.
// No memory clobber, though it writes LDS: the products and fragment reads around it stay free to move, and what keeps an LDS
// read from crossing the write of its stage are the clobbers of the two waits below alone - every stage is read between
// the wait_vm_barrier that says it has arrived and the wait_lds_barrier (or next wait_vm_barrier) that hands it back.
__device__ __forceinline__ void dma_1k(uint32_t lds_addr, int voff, u32x4_t rsrc, int soff) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "{m0}"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff));
}

// at most N of this wavefront's loads still in flight and all its LDS reads returned, then the workgroup's barrier
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// all LDS reads of this wavefront returned, then the barrier; loads stay in flight
__device__ __forceinline__ void wait_lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// buffer descriptor over `bytes` bytes from `base`
template <typename T>
__device__ __forceinline__ u32x4_t make_rsrc(const T* base, int64_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return u32x4_t{static_cast<uint32_t>(a), static_cast<uint32_t>(a >> 32) & 0xffffu,
                   static_cast<uint32_t>(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000u};
}

__device__ __forceinline__ uint32_t lds_address(const char* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}

}  // namespace
}  // namespace freemi
