// What the E2M3 GEMM kernels share: the operand format's sizes, the transfers from global memory into LDS, a product's arguments.
#pragma once
#include "qvggt_common.h"

#include <type_traits>
#include <utility>

namespace qvggt {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int U_BYTES = 48;        // bytes per row per unit: 64 codes of 6 bits
constexpr int RB = 128;            // rows per block of the operand format
constexpr int RB_BYTES = RB * U_BYTES;   // one unit of one block: 6 KiB contiguous
constexpr int RB_PIECES = RB_BYTES / 1024;
// Scale operands of the matrix builtin.  Constant zeros make the compiler emit the instruction form without block scales
// (v_mfma_f32_32x32x64_f8f6f4: products as they are), one instruction per MFMA instead of two; 0x7F7F7F7F (E8M0 exponent 127 = 2^0
// in every byte) is the explicit unit scale and gives the same sums.
constexpr int UNIT_SCALE_ONE = 0;

// Global memory -> LDS, 16 bytes per lane: lane l reads base + lane_off and writes LDS address lds_base + 16 * l.  M0 carries the
// LDS base; each transfer sets it itself and says so, so nothing depends on what the compiler does with that register elsewhere.  A transfer wants
// one wait state behind a scalar write of M0, which the compiler does not put inside an asm block (0.1 % of a GEMM's time).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void e_dma16(uint32_t lane_off, const void *base, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_base) : "memory", "m0");
}
// 4 bytes per lane: lane l writes lds_base + 4 * l
__device__ inline void e_dma4(const void *src, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds_base) : "memory", "m0");
}
#pragma clang diagnostic pop
template <class F, int... Is>
__device__ inline void e_static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ inline void e_static_for(F &&f)
{
    e_static_for_impl(f, std::make_integer_sequence<int, N>{});
}
template <int N>
__device__ inline void e_wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A product's operands and result; xzero and wsum only with SHIFTED codes.
struct E2m3Problem {
    const uint8_t *Xf;
    const float *sx;
    const uint8_t *Wf;
    const float *sw;
    const uint16_t *bias;
    int M, N, K;
    uint16_t *Y;
    int32_t *acc_debug;
    const float *xzero, *wsum;

    // token rows row0 .. row0 + rows - 1; row0 is a multiple of 128, i.e. whole blocks of the operand format
    E2m3Problem part(int row0, int rows) const
    {
        E2m3Problem p = *this;
        p.Xf += (size_t)row0 * ((size_t)K / 4 * 3);
        p.sx += row0;
        p.M = rows;
        p.Y += (size_t)row0 * N;
        if (acc_debug != nullptr) p.acc_debug += (size_t)row0 * N;
        if (xzero != nullptr) p.xzero += row0;
        return p;
    }
};

}  // namespace qvggt
