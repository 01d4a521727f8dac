// Transfers from global memory straight into LDS.  M0 carries the LDS base; every transfer sets it itself and names it as clobbered, so nothing depends
// on what the compiler does with that register between two of them.  A transfer wants one wait state behind a scalar write of M0, which the
// compiler does not put inside an asm block: the s_nop (0.1 % of a GEMM's time).
// The global address is a wave-uniform 64-bit base (scalar registers) plus a 32-bit offset per lane: moving along K only touches the
// scalar base, no vector ALU work.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace qvggt {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane: lane l writes lds_base + OFF + 16 * l.  The instruction offset of such a transfer moves the LDS address and
// the global address alike: with one LDS base, transfers to different places of a stage differ only in OFF (the lane's global
// offset is pre-compensated by -OFF).
template <int OFF = 0>
__device__ inline void dma16(uint32_t lane_off, const void *base, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(lane_off), "s"(base), "s"(lds_base), "n"(OFF) : "memory", "m0");
}
// the same to lds_base + AT, the global address as it is
template <int AT>
__device__ inline void dma16_at(uint32_t lane_off, const void *base, uint32_t lds_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_base), "n"(AT) : "memory", "m0", "scc");
}
// 4 bytes per lane, from an address of its own: lane l writes lds_base + 4 * l
__device__ inline void dma4(const void *src, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds_base) : "memory", "m0");
}
__device__ inline void dma4(uint32_t lane_off, const void *base, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_base) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace qvggt
