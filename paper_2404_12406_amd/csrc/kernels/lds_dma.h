// Buffer descriptors, LDS-DMA loads and the waits that order them, shared by
// the GEMM kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ms {
namespace g2 {

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}

// One 16-byte LDS-DMA load: lane l's 16 bytes from byte offset `off` of the
// buffer land at lds + 16 l (M0 holds the wave's LDS base).
//
// Contractions with an M/N-contiguous operand (ASM = true) issue it through
// inline assembly so that the compiler does not track it: for a pending
// LDS-DMA load the compiler puts a wait for every outstanding vector-memory
// operation in front of each transposing LDS read (ds_read_b64_tr_b16),
// which drains all refill loads in flight at every slice.  The others keep
// the builtin, whose loads the scheduler can spread between the MFMAs.
// Ordering in the assembly form is the kernel's own:
//  * completion: its vmcnt waits before each barrier;
//  * a refill writes a stage no wave reads until after the next barrier, and
//    a volatile asm statement never moves across the barrier;
//  * block_sync() tells the compiler that LDS may have changed, so no LDS
//    value read before a barrier is reused after it.
// M0 is reserved by the compiler and no other instruction of these kernels
// reads it.  A load that writes LDS needs one wait state after a scalar write of
// M0; the compiler puts it there for the builtin but does not look inside
// inline assembly, so the assembly forms carry their own s_nop.
// (The offset is computed into a named value first: passing a conditional
// expression straight into the builtin inside a kernel template makes the
// host pass drop the kernel's launch stub.)
template <bool ASM>
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, char *lds, uint32_t off) {
    if constexpr (ASM) {
        const uint32_t base = (uint32_t)(uintptr_t)(lds_void_t *)lds;
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds" ::"v"(off), "s"(base), "s"(r));
    } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t *)lds, 16, off, 0, 0, 0);
    }
}

// The assembly form with a uniform byte offset added to every lane's, and its
// 4-byte sibling (lane l's dword lands at lds + 4 l).
__device__ __forceinline__ void dma16s(__amdgpu_buffer_rsrc_t r, char *lds, uint32_t off, uint32_t soff) {
    const uint32_t base = (uint32_t)(uintptr_t)(lds_void_t *)lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, %3 offen lds" ::"v"(off), "s"(base), "s"(r), "s"(soff));
}
__device__ __forceinline__ void dma4s(__amdgpu_buffer_rsrc_t r, char *lds, uint32_t off, uint32_t soff) {
    const uint32_t base = (uint32_t)(uintptr_t)(lds_void_t *)lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dword %0, %2, %3 offen lds" ::"v"(off), "s"(base), "s"(r), "s"(soff));
}

// Workgroup barrier; with untracked LDS-DMA loads it is also a compiler-level
// memory fence (the barrier builtin alone does not stop the compiler from
// keeping LDS values across it).
template <bool ASM>
__device__ __forceinline__ void block_sync() {
    if constexpr (ASM) __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    if constexpr (ASM) __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt[3:0] | [15:14],
// expcnt[6:4] = 7, lgkmcnt[11:8] = 15).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xc07f); }

}  // namespace g2
}  // namespace ms
