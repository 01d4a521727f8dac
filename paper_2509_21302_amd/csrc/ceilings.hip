// Measurement helper of the benchmark: register-only loops of the matrix instructions that the GEMMs of many tokens are built on, so that a
// run can state, beside the published peak, what the matrix pipes deliver on this board when nothing has to be fed to them
// (one wave per SIMD, 32 independent 16x16 accumulators, operands that stay in registers).  No memory traffic.
// Operands are codes of a normal distribution, as quantized rows have: the power limit is what the loop runs into, and random bits draw more.
#include "qvggt_common.h"

namespace qvggt {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// roughly N(0, 1): the sum of a hash's four bytes
__device__ inline float normal_of(uint32_t n)
{
    n ^= n >> 16; n *= 0x7FEB352Du; n ^= n >> 15; n *= 0x846CA68Bu; n ^= n >> 16;
    return ((float)((n & 255) + (n >> 8 & 255) + (n >> 16 & 255) + (n >> 24)) - 510.0f) * (1.0f / 147.8f);
}
// 16 int8 codes, a quarter of the absmax wide (8-bit codes of normal rows)
__device__ __forceinline__ v4i int8_codes(uint32_t seed)
{
    v4i f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t w = 0;
        for (int b = 0; b < 4; ++b) w |= ((uint32_t)(int)rintf(normal_of(seed + e * 4 + b) * 32.0f) & 255u) << (8 * b);
        f[e] = (int)w;
    }
    return f;
}
// 32 E2M3 numbers of the codes -7 .. 7
__device__ __forceinline__ v8i e2m3_codes(uint32_t seed)
{
    constexpr uint64_t MAG = 0x00ull | (0x08ull << 5) | (0x10ull << 10) | (0x14ull << 15) | (0x18ull << 20) | (0x1Aull << 25) | (0x1Cull << 30) | (0x1Eull << 35);
    uint64_t w[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const int q = (int)fminf(fmaxf(rintf(normal_of(seed + i) * 2.2f), -7.0f), 7.0f);
        const uint64_t field = (MAG >> (5 * abs(q)) & 31) | (q < 0 ? 32u : 0u);
        w[6 * i / 64] |= field << (6 * i % 64);
        if (6 * i % 64 > 58) w[6 * i / 64 + 1] |= field >> (64 - 6 * i % 64);
    }
    return v8i{(int)w[0], (int)(w[0] >> 32), (int)w[1], (int)(w[1] >> 32), (int)w[2], (int)(w[2] >> 32), 0, 0};
}

// KIND 0: v_mfma_i32_16x16x64_i8 (int8 blocks); KIND 1: v_mfma_f32_16x16x128_f8f6f4 on E2M3 operands
template <int KIND>
__global__ __launch_bounds__(256, 1) void mfma_ceiling_kernel(int iters, float *__restrict__ sink)
{
    constexpr int NA = 8, NB = 4;
    const uint32_t seed = (blockIdx.x * 256 + threadIdx.x) * 512u;
    float total = 0.0f;
    auto run = [&](auto codes, auto multiply, auto zero) {
        decltype(codes(0u)) A[NA], B[NB];
#pragma unroll
        for (int f = 0; f < NA; ++f) A[f] = codes(seed + f * 32);
#pragma unroll
        for (int f = 0; f < NB; ++f) B[f] = codes(seed + (NA + f) * 32);
        decltype(zero) acc[NA][NB];
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b] = zero;
        for (int it = 0; it < iters; ++it) {
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    acc[a][b] = multiply(A[a], B[b], acc[a][b]);
                    __builtin_amdgcn_sched_barrier(0);               // as they stand: reordered, the compiler moves accumulators between them
                }
        }
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) total += (float)acc[a][b][r];
    };
    if constexpr (KIND == 0) run(int8_codes, [](v4i a, v4i b, v4i s) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, s, 0, 0, 0); }, v4i{0, 0, 0, 0});
    else run(e2m3_codes, [](v8i a, v8i b, v4f s) { return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, s, 2, 2, 0, 0, 0, 0); }, v4f{0, 0, 0, 0});
    sink[blockIdx.x * 256 + threadIdx.x] = total;
}

hipError_t run_mfma_ceiling(int kind, int iters, float *sink, hipStream_t stream)
{
    if (kind == 0) mfma_ceiling_kernel<0><<<256, 256, 0, stream>>>(iters, sink);
    else mfma_ceiling_kernel<1><<<256, 256, 0, stream>>>(iters, sink);
    return hipGetLastError();
}

}  // namespace qvggt
