// What the E2M3 GEMM kernels share: the operand format's sizes, a product's arguments.
#pragma once
#include "lds_transfer.h"
#include "qvggt_common.h"

#include <type_traits>
#include <utility>

namespace qvggt {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int U_BYTES = 48;        // bytes per row per unit: 64 codes of 6 bits
constexpr int RB = 128;            // rows per block of the operand format
constexpr int RB_BYTES = RB * U_BYTES;   // one unit of one block: 6 KiB contiguous
constexpr int RB_PIECES = RB_BYTES / 1024;
// Scale operands of the matrix builtin.  Constant zeros make the compiler emit the instruction form without block scales
// (v_mfma_f32_32x32x64_f8f6f4: products as they are), one instruction per MFMA instead of two; 0x7F7F7F7F (E8M0 exponent 127 = 2^0
// in every byte) is the explicit unit scale and gives the same sums.
constexpr int UNIT_SCALE_ONE = 0;

template <class F, int... Is>
__device__ __attribute__((always_inline)) inline void e_static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __attribute__((always_inline)) inline void e_static_for(F &&f)
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

// Tiles of 256 tokens x 256 channels (gemm_e2m3_256.hip), where e2m3_tiles256 says so.
template <bool SHIFTED>
hipError_t run_e2m3_256(const E2m3Problem &p, hipStream_t stream);

}  // namespace qvggt
