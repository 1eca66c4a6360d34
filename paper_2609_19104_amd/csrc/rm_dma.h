// Loads straight from memory into LDS, shared by the kernels that stage matrix-core operands this way: 64-column bf16
// stages, whose rows (128 bytes) are kept as eight 16-byte pieces, piece p of row r at position p ^ row_swz(r), so
// that fragment reads (16 rows at one piece) hit distinct LDS banks, both with 32 banks served 8 lanes a cycle and with
// 64 banks served 16 lanes a cycle.
#pragma once

#include "rm_internal.h"

namespace rm_dma {

constexpr int kStageK = 64;             // columns per stage
constexpr int kRowBytes = kStageK * 2;

__device__ __forceinline__ int row_swz(int r) { return (r ^ (r >> 3)) & 7; }  // r: row mod 16

// One load of 16 bytes per lane into LDS at lds + 16 lane (M0 holds the wave's LDS base while it issues; M0 is
// the compiler's register, so its value is kept and put back).  Issued as inline assembly so that the compiler,
// which cannot tell the stage buffers apart, adds no wait of its own for it before the LDS reads: the waits are
// the explicit ones below.
__device__ __forceinline__ void dma16(const void *g, uint32_t lds) {
    uint32_t keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(g), "s"(lds)
        : "memory");
}

// Wait until at most N of this wave's vector-memory operations are in flight and all its LDS operations are
// done, then the workgroup barrier.  The compiler may not move memory accesses across it.
template <int N>
__device__ __forceinline__ void wait_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ uint32_t lds_addr(const uint8_t *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) uint8_t *)p));
}

}  // namespace rm_dma
