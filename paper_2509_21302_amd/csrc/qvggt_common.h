// Shared device-side helpers of the qvggt HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qvggt {

constexpr int kWave = 64;
constexpr int kMinK = 128;
constexpr int kMaxK = 8192;
// A quantization step below the smallest normal fp32 number (2^-126) counts as 0: the row gets step 0 and codes 0 (a dynamic
// step), or codes 0 (a given one).  Such a step could not be inverted in fp32 (7 / absmax would overflow).
constexpr float kMinStep = 1.17549435e-38f;

// Width argument of the quantizing launchers: 4 = 4-bit codes packed two per byte; kInt8Container + b = b-bit codes
// (4 <= b <= 8) stored one per byte as int8 (so that weights and activations of one int8 GEMM may take different widths)
constexpr int kInt8Container = 32;
inline int code_width(int bits) { return bits >= kInt8Container ? bits - kInt8Container : bits; }

// Position of natural element e inside a packed row of K codes.  Two codes share a byte:
// position p lives in byte p / 2, low nibble when p is even.  The same map is used for
// activations and weights, so integer dot products do not depend on it.
//
// For K = 1024, 2048, 4096 the map is the one the matrix-core rotation kernel produces
// naturally: with e = 128*hb + 32*nt + c (c < 32, nt < 4), position = c*(K/32) + nt + 4*hb',
// where hb' = hb except for K = 4096, which swaps bits 3 and 4 of hb.  Other K keep natural order.
__host__ __device__ inline bool layout_is_permuted(int K) { return K == 1024 || K == 2048 || K == 4096; }

__host__ __device__ inline int swap_bits_3_4(int v) { return (v & ~0x18) | ((v & 8) << 1) | ((v & 16) >> 1); }

__host__ __device__ inline int code_position(int e, int K)
{
    if (!layout_is_permuted(K)) return e;
    int c = e & 31, nt = (e >> 5) & 3, hb = e >> 7;
    if (K == 4096) hb = swap_bits_3_4(hb);
    return c * (K / 32) + nt + 4 * hb;
}
// Inverse of code_position: the natural element stored at position p.
__host__ __device__ inline int code_element(int p, int K)
{
    if (!layout_is_permuted(K)) return p;
    int c = p / (K / 32), l = p % (K / 32);
    int nt = l & 3, hb = l >> 2;
    if (K == 4096) hb = swap_bits_3_4(hb);
    return 128 * hb + 32 * nt + c;
}

__device__ inline float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// two floats -> packed bf16 pair (round to nearest even), lo in bits 0..15
__device__ inline uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    bf2 p;
    p[0] = (__bf16)lo;
    p[1] = (__bf16)hi;
    return *reinterpret_cast<uint32_t *>(&p);
}

// Lanes of one wave hand data to each other through a wave-private LDS area.  LDS operations of a wave execute in order, so
// no instruction has to separate the writes from the reads; the compiler, however, must be told that a lane is about to
// read what other lanes wrote (it may otherwise treat such a read as a repeat of an earlier one).
__device__ inline void lanes_exchange_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Maximum over groups of lanes without going through LDS: four DPP steps inside a row of 16 lanes (quad permutes, then
// mirrors: after each step every lane of the group holds the group's maximum), then the gfx950 row swaps across rows.
template <int CTRL>
__device__ inline float dpp_max_step(float v)
{
    const int p = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false);
    return fmaxf(v, __int_as_float(p));
}
__device__ inline float max_over_16_lanes(float v)
{
    v = dpp_max_step<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v = dpp_max_step<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    v = dpp_max_step<0x141>(v);    // row_half_mirror
    v = dpp_max_step<0x140>(v);    // row_mirror
    return v;
}
__device__ inline float max_over_32_lanes(float v)   // lanes 0..31 and lanes 32..63 separately
{
    v = max_over_16_lanes(v);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float max_over_64_lanes(float v)
{
    v = max_over_32_lanes(v);
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The six Walsh-Hadamard butterflies over the lane bits, for R registers that each hold one value per lane: x[l] becomes
// x[l] + x[l ^ m] in lanes without bit m and x[l ^ m] - x[l] in the others.  Lane bits 0 .. 3 by DPP (quad permutes; 4 = a half-row
// mirror of a quad reversal; 8 = a rotation of the row of 16), the sign in the multiplier of an exact fma.  Bits 4 and 5 by row swaps of
// register pairs: swapped, the pair holds the two partners of each butterfly, and a second swap puts the results back.  No LDS:
// six cross-lane reads per value through it were what the row kernels spent their time on.
template <int CTRL>
__device__ inline float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int R>
__device__ inline void lane_butterflies(float (&x)[R], int lane)
{
    static_assert(R % 2 == 0, "the row swaps work on pairs of registers");
    const float s1 = (lane & 1) ? -1.0f : 1.0f, s2 = (lane & 2) ? -1.0f : 1.0f, s4 = (lane & 4) ? -1.0f : 1.0f, s8 = (lane & 8) ? -1.0f : 1.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        x[r] = fmaf(x[r], s1, dpp_move<0xB1>(x[r]));
        x[r] = fmaf(x[r], s2, dpp_move<0x4E>(x[r]));
        x[r] = fmaf(x[r], s4, dpp_move<0x141>(dpp_move<0x1B>(x[r])));
        x[r] = fmaf(x[r], s8, dpp_move<0x128>(x[r]));
    }
#pragma unroll
    for (int r = 0; r < R; r += 2) {
        auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[r]), __float_as_uint(x[r + 1]), false, false);
        float a = __uint_as_float(p[0]), b = __uint_as_float(p[1]);
        p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a + b), __float_as_uint(a - b), false, false);
        p = __builtin_amdgcn_permlane32_swap(p[0], p[1], false, false);
        a = __uint_as_float(p[0]); b = __uint_as_float(p[1]);
        p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a + b), __float_as_uint(a - b), false, false);
        x[r] = __uint_as_float(p[0]);
        x[r + 1] = __uint_as_float(p[1]);
    }
}

// The two butterflies over the wave number (0 .. 3) of a row that four waves of a block share, through LDS [4][R / 4][64] float4:
// every wave leaves its values and adds up the four of each position.  Ends with a barrier: the area may be written again.
template <int R>
__device__ inline void wave_butterflies(float (&x)[R], float4 *area, int sub, int lane)
{
    static_assert(R % 4 == 0, "values move four at a time");
#pragma unroll
    for (int q = 0; q < R / 4; ++q) area[(sub * (R / 4) + q) * 64 + lane] = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
    __syncthreads();
    const float s1 = (sub & 1) ? -1.0f : 1.0f, s2 = (sub & 2) ? -1.0f : 1.0f;
    auto sum = [&](float a, float b, float c, float d) { return fmaf(s2, fmaf(s1, d, c), fmaf(s1, b, a)); };
#pragma unroll
    for (int q = 0; q < R / 4; ++q) {
        const float4 a = area[q * 64 + lane], b = area[(R / 4 + q) * 64 + lane], c = area[(2 * (R / 4) + q) * 64 + lane], d = area[(3 * (R / 4) + q) * 64 + lane];
        x[4 * q] = sum(a.x, b.x, c.x, d.x);
        x[4 * q + 1] = sum(a.y, b.y, c.y, d.y);
        x[4 * q + 2] = sum(a.z, b.z, c.z, d.z);
        x[4 * q + 3] = sum(a.w, b.w, c.w, d.w);
    }
    __syncthreads();
}
// maximum over the four waves of a block (v the same in all lanes of a wave); red[4] is free again after the next barrier
__device__ inline float max_over_4_waves(float v, float *red)
{
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// Adding it rounds a float of magnitude < 2^22 to the nearest integer (ties to even) and leaves that integer, two's complement, in the
// low bits of the sum's pattern.
constexpr float kRoundMagic = 12582912.0f;      // 1.5 * 2^23

// Sum over all 64 lanes, the same butterflies with an add (every lane ends with the total).
template <int CTRL>
__device__ inline float dpp_add_step(float v)
{
    const int p = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false);
    return v + __int_as_float(p);
}
__device__ inline float sum_over_64_lanes(float v)
{
    v = dpp_add_step<0xB1>(v);
    v = dpp_add_step<0x4E>(v);
    v = dpp_add_step<0x141>(v);
    v = dpp_add_step<0x140>(v);
    const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
}

// LayerNorm in front of the rotation (optional): y = (x - mean) / sqrt(var + eps) * gamma + beta over the K channels of a token.
// gamma / beta may be nullptr (1 / 0).  on == 0: no normalisation.
struct LnParams {
    const float *gamma;
    const float *beta;
    float eps;
    int on;
};

// Kernels that need more dynamic LDS than a launch gets by default.  Each source file that has such kernels lists them in a
// static LdsKernels object (filled when the library is loaded; no HIP call is made then).  prepare_device() raises the limit of
// every listed kernel on the calling thread's current device the first time it runs there (and resolves the address of the
// library's own workspace on that device); later calls are one atomic load.  Thread-safe; qvggt_init() is its public form.
struct LdsKernel {
    const void *fn;
    int lds_bytes;
};
void register_lds_kernels(const LdsKernel *list, int n);
struct LdsKernels {
    template <int N>
    explicit LdsKernels(const LdsKernel (&list)[N]) { register_lds_kernels(list, N); }
};
hipError_t prepare_device(int *device = nullptr);

}  // namespace qvggt
