// Copies from memory to LDS past the registers, and the barrier that goes
// with them (kernels with fixed operand slots in LDS).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace bsm {

// The compiler does not count these copies; wait_dma() waits for the wave's own.
__device__ inline void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroup barrier: the wave's own LDS reads are done before it, nothing
// moves across it.
__device__ inline void group_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// PIECES consecutive 16-byte pieces from src (16-byte aligned) to the LDS
// address `slot`: 64 a copy, the lanes' bytes consecutive at m0.
// voff = 16 lane; every lane of the wave is active, the last copy runs with
// the lanes it needs.  The five wait states cover a source address that a
// lane read has just written; M0 is declared as written, EXEC is as before.
template <int PIECES>
__device__ inline void stage_pieces(uint64_t src, uint32_t slot, uint32_t voff) {
    constexpr int FULL = PIECES / 64, REST = PIECES % 64;
#pragma unroll
    for (int q = 0; q < FULL / 4; ++q)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "global_load_lds_dwordx4 %1, %2\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:1024\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:2048\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:3072"
                     :: "s"(slot + 4096 * q), "v"(voff + 4096 * q), "s"(src) : "m0", "memory");
#pragma unroll
    for (int q = FULL / 4 * 4; q < FULL; ++q)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                     "global_load_lds_dwordx4 %1, %2"
                     :: "s"(slot + 1024 * q), "v"(voff + 1024 * q), "s"(src) : "m0", "memory");
    if constexpr (REST > 0)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\ts_mov_b64 exec, %3\n\t"
                     "global_load_lds_dwordx4 %1, %2\n\t"
                     "s_mov_b64 exec, -1"
                     :: "s"(slot + 1024 * FULL), "v"(voff + 1024 * FULL), "s"(src),
                        "s"((1ull << REST) - 1) : "m0", "memory");
}

// The same with a number of pieces known at run time.
__device__ inline void stage_pieces(uint64_t src, uint32_t slot, int pieces, uint32_t voff) {
    for (int p = 0; p < pieces; p += 64) {
        const uint64_t ex = pieces - p >= 64 ? ~0ull : (1ull << (pieces - p)) - 1ull;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\ts_mov_b64 exec, %3\n\t"
                     "global_load_lds_dwordx4 %1, %2\n\t"
                     "s_mov_b64 exec, -1"
                     :: "s"(slot + p * 16), "v"(voff + p * 16), "s"(src), "s"(ex) : "m0", "memory");
    }
}

// 16 bytes a lane from src + voff to consecutive LDS bytes at `slot`, past
// the registers.
__device__ inline void dma16(uint32_t slot, uint32_t voff, const double *src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(slot), "v"(voff), "s"(reinterpret_cast<uint64_t>(src)) : "m0", "memory");
}

}  // namespace bsm
