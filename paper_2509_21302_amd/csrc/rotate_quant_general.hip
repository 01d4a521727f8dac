// Online kernel 1 and its offline twins for input sizes that are not powers of two: K = 2^n * m with m = 12, 20 or 28
// (paper Sec. 3.2: H_K = H_{2^n} (x) H_m).  H_m is Paley's Hadamard matrix (type I from GF(11) and GF(19), type II from
// GF(13)); its entries are computed at compile time from the quadratic residues, so the m-point stage is straight-line
// adds and subtracts.  Element e = a * m + b (a < 2^n, b < m); a wavefront owns a row, lane l holds the m values of every
// a = l + 64 * c: the m-point transform is inside a lane, the six low bits of a go through cross-lane exchanges, the
// remaining bits are register-to-register butterflies.  Codes are written in natural order (element e -> position e).
// This is the general path: VGGT-1B itself has no layer that needs it, and bf16 activations of m = 12, and m = 20 but for K = 1280, are quantized in
// rotate_quant_paley.hip.  Bound by the vector ALU (34350 x 768 bf16: 38 us with dense m-point sums and the lane bits through LDS, 28 us now).
#include "paley.h"
#include "qvggt_common.h"
#include "rotate_rows.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace qvggt {

namespace gen {

// Inputs 4 g .. 4 g + 3 of output c, up to the sign of the first: which of the sums x0 +- x1 +- (x2 +- x3) they make (bit 0: x1 subtracted,
// bit 1: x3 against x2, bit 2: x2 against x0)
template <int MM>
constexpr int sum_of_four(int g, int c)
{
    const int s0 = paley_entry<MM>(4 * g, c), s1 = paley_entry<MM>(4 * g + 1, c), s2 = paley_entry<MM>(4 * g + 2, c), s3 = paley_entry<MM>(4 * g + 3, c);
    return (s0 * s1 < 0 ? 1 : 0) | (s2 * s3 < 0 ? 2 : 0) | (s0 * s2 < 0 ? 4 : 0);
}
// After group g, is it the negative of output c's partial sum that is held?  (It is while every group so far entered with a minus.)
template <int MM>
constexpr bool partial_is_negated(int g, int c)
{
    for (int k = 0; k <= g; ++k)
        if (paley_entry<MM>(4 * k, c) > 0) return false;
    return true;
}

template <class F, int... Is>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

enum Mode { kQuantize = 0, kColAbsMax = 1 };

// Four waves per row at K = 5120 and 6144: with one, a row and its multipliers take more than the 256 registers of a wave that shares
// its SIMD.  34350 rows (bf16): 667 and 817 us with one wave per row.
constexpr int waves_per_row(int n2, int mm) { return n2 / 64 * mm >= 80 ? 4 : 1; }

}  // namespace gen

// mul_mode 0: mul[j] used as given (inv_smooth, or 1/sqrt(K) when mul == nullptr); 1: 1 / (K * mul[j]) (weights)
// CB: bits a stored code occupies (4 or 8; 6: 4-bit codes as E2M3 blocks, dynamic steps); qmax: largest code; step: static quantization step or nullptr
// BOTH (CB = 6): the codes also go out as rows of packed nibbles, to rows_out
template <int N2, int MM, bool F32, int MODE, int CB, bool BOTH = false>
__global__ __launch_bounds__(256) void rotate_rows_general_kernel(const void *__restrict__ X, int rows,
                                                                  const int8_t *__restrict__ signs,
                                                                  const float *__restrict__ mul, int mul_mode,
                                                                  uint8_t *__restrict__ packed, float *__restrict__ scale,
                                                                  unsigned int *__restrict__ col_absmax_bits,
                                                                  const float *__restrict__ step, int step_stride, float qmax,
                                                                  uint8_t *__restrict__ rows_out = nullptr)
{
    // waves per row: one, or the four of a block where a row would take 80 registers of a lane or more (see gen::waves_per_row).  A wave then
    // has N2 / 4 consecutive values of a, and two butterflies go over the wave number.
    constexpr int K = N2 * MM, WPR = gen::waves_per_row(N2, MM), C = N2 / WPR / 64, R = C * MM;
    static_assert(N2 / WPR >= 64 && (N2 & (N2 - 1)) == 0, "the power-of-two factor covers the 64 lanes");
    const int lane = threadIdx.x & 63;
    const int sub = WPR > 1 ? (int)(threadIdx.x >> 6) : 0, first = sub * (K / WPR);       // this wave's part of a row
    constexpr bool E2M3 = (CB == 6);
    const int group = !E2M3 || WPR == 1 || rows > kFewSharedRows ? kE2m3Group : 1;       // rows that leave together
    const int wave = WPR > 1 ? (int)blockIdx.x * (E2M3 ? group : 1) : (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int nwaves = WPR > 1 ? (int)gridDim.x : (int)gridDim.x * 4;
    __shared__ float4 exchange[WPR > 1 ? K / 4 : 1];
    __shared__ float red[4];
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[E2M3 ? E2m3Stage<K>::BYTES : 16];

    // per-lane constants: register r = c * MM + b holds element e = (lane + 64 c) * MM + b
    constexpr bool SIGN_MASKS = R <= 32;       // signs as masks while there is room, one bit per register otherwise
    float cm[R];
    uint32_t neg[SIGN_MASKS ? R : (R + 31) / 32];
#pragma unroll
    for (int w = 0; w < (SIGN_MASKS ? R : (R + 31) / 32); ++w) neg[w] = 0;
    const float rs = 1.0f / sqrtf((float)K);
    // loads first (all in flight together), arithmetic afterwards
    if (signs != nullptr) {
        int8_t sb[R];
#pragma unroll
        for (int r = 0; r < R; ++r) sb[r] = signs[first + (lane + 64 * (r / MM)) * MM + (r % MM)];
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (sb[r] < 0) neg[SIGN_MASKS ? r : r >> 5] |= SIGN_MASKS ? 0x80000000u : 1u << (r & 31);
    }
    if (mul != nullptr) {
#pragma unroll
        for (int r = 0; r < R; ++r) cm[r] = mul[first + (lane + 64 * (r / MM)) * MM + (r % MM)];
        if (mul_mode) {
#pragma unroll
            for (int r = 0; r < R; ++r) cm[r] = 1.0f / ((float)K * cm[r]);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) cm[r] = rs;
    }

    float colmax[MODE == gen::kColAbsMax ? R : 1];
#pragma unroll
    for (int r = 0; r < (MODE == gen::kColAbsMax ? R : 1); ++r) colmax[r] = 0.0f;
    // E2M3: a block takes a group of consecutive rows at a time, one per wave or (WPR > 1) one after the other; past the end: the last row, not
    // written
    const int last = group - 1;
    for (int row = wave; (E2M3 ? row & ~last : row) < rows; row += !(E2M3 && WPR > 1) ? nwaves : (row & last) == last ? group * nwaves - last : 1) {
        float x[R];
        // a lane's MM values of one a are contiguous: 8-byte (bf16) or 16-byte (f32) pieces of four values
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const size_t e0 = (size_t)(E2M3 ? min(row, rows - 1) : row) * K + first + (size_t)(lane + 64 * c) * MM;
#pragma unroll
            for (int q = 0; q < MM / 4; ++q) {
                if constexpr (F32) {
                    const float4 v = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(X) + e0 + 4 * q);
                    x[c * MM + 4 * q] = v.x; x[c * MM + 4 * q + 1] = v.y; x[c * MM + 4 * q + 2] = v.z; x[c * MM + 4 * q + 3] = v.w;
                } else {
                    const uint2 v = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(X) + e0 + 4 * q);
                    x[c * MM + 4 * q] = __uint_as_float(v.x << 16); x[c * MM + 4 * q + 1] = __uint_as_float(v.x & 0xFFFF0000u);
                    x[c * MM + 4 * q + 2] = __uint_as_float(v.y << 16); x[c * MM + 4 * q + 3] = __uint_as_float(v.y & 0xFFFF0000u);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            x[r] = __uint_as_float(__float_as_uint(x[r]) ^ (SIGN_MASKS ? neg[r] : (neg[r >> 5] << (31 - (r & 31))) & 0x80000000u));

        // H_m inside every group of MM registers: y[b'] = sum_b x[b] H[b][b'], signs known at compile time.  The inputs are taken four at a
        // time: up to a sign, an output needs one of the eight sums x0 +- x1 +- x2 +- x3, which cost twelve additions together and are
        // shared by all outputs; an output adds MM / 4 of them.  5, 7 and 9 operations per element for m = 12, 20 and 28 instead of m.
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float y[MM];
            gen::static_for<MM / 4>([&](auto g_c) {
                constexpr int g = decltype(g_c)::value;
                const float *in = x + c * MM + 4 * g;
                const float p[2] = {in[0] + in[1], in[0] - in[1]}, q[2] = {in[2] + in[3], in[2] - in[3]};
                float t[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = (k & 4) ? p[k & 1] - q[(k >> 1) & 1] : p[k & 1] + q[(k >> 1) & 1];
                gen::static_for<MM>([&](auto bp_c) {
                    constexpr int bp = decltype(bp_c)::value;
                    const float v = t[gen::sum_of_four<MM>(g, bp)];
                    constexpr bool minus = gen::paley_entry<MM>(4 * g, bp) < 0;
                    // y[bp] holds the partial sum, or its negative (known at compile time)
                    if constexpr (g == 0) y[bp] = v;
                    else if constexpr (gen::partial_is_negated<MM>(g - 1, bp) == minus) y[bp] += v;
                    else if constexpr (minus) y[bp] -= v;
                    else y[bp] = v - y[bp];
                });
            });
            gen::static_for<MM>([&](auto bp_c) {
                constexpr int bp = decltype(bp_c)::value;
                x[c * MM + bp] = gen::partial_is_negated<MM>(MM / 4 - 1, bp) ? -y[bp] : y[bp];
            });
        }
        // H_{2^n} over a = lane + 64 c: the six lane bits, then the bits of c
        lane_butterflies(x, lane);
#pragma unroll
        for (int h = 1; h < C; h <<= 1)
#pragma unroll
            for (int c = 0; c < C; ++c)
                if ((c & h) == 0) {
#pragma unroll
                    for (int b = 0; b < MM; ++b) {
                        const float a = x[c * MM + b], d = x[(c + h) * MM + b];
                        x[c * MM + b] = a + d;
                        x[(c + h) * MM + b] = a - d;
                    }
                }

        if constexpr (WPR > 1) wave_butterflies(x, exchange, sub, lane);
        float amax = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) { x[r] *= cm[r]; amax = fmaxf(amax, fabsf(x[r])); }

        if constexpr (MODE == gen::kColAbsMax) {
            // the wave keeps a running maximum over its rows; one atomic per column after the loop
#pragma unroll
            for (int r = 0; r < R; ++r) colmax[r] = fmaxf(colmax[r], fabsf(x[r]));
        } else {
            float inv, delta;
            if (step != nullptr) {
                delta = step[(size_t)row * step_stride];
                inv = delta >= kMinStep ? 1.0f / delta : 0.0f;
            } else {
                amax = max_over_64_lanes(amax);
                if constexpr (WPR > 1) amax = max_over_4_waves(amax, red);
                const bool live = amax >= qmax * kMinStep;
                delta = live ? amax / qmax : 0.0f;
                inv = live ? qmax / amax : 0.0f;
            }
            if (lane == 0 && sub == 0 && (!E2M3 || row < rows)) scale[row] = delta;
            const int q_hi = (int)qmax, q_lo = -q_hi - 1;
            // a step from the row's own maximum bounds |x * inv| by qmax (1 + 2^-22): rounding cannot leave the range, and the code is the low
            // bits of one fma.  (inv is 0 for a row without a step, or whose values overflowed: the general form gives codes 0 there.)
            const bool bounded = step == nullptr && inv > 0.0f;
            auto code_of = [&](int r) -> uint32_t {       // two's complement in the low CB bits, anything above
                return bounded ? __float_as_uint(fmaf(x[r], inv, kRoundMagic)) : (uint32_t)min(q_hi, max(q_lo, (int)__builtin_rintf(x[r] * inv)));
            };
            if constexpr (E2M3) {
                uint8_t *stage = lds_stage + (row & last) * E2m3Stage<K>::PITCH + first;
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int g = 0; g < MM; g += 4)
                        *reinterpret_cast<uint32_t *>(stage + (lane + 64 * c) * MM + g) = low_bytes(code_of(c * MM + g), code_of(c * MM + g + 1), code_of(c * MM + g + 2), code_of(c * MM + g + 3));
                if (WPR == 1 || (row & last) == last) {       // the same for the whole block
                    __syncthreads();
                    flush_e2m3<K, BOTH>(lds_stage, row & ~last, group, rows, packed, rows_out);
                    __syncthreads();
                }
                continue;
            }
            uint8_t *out = packed + (size_t)row * (K * CB / 8);
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int g = 0; g < MM / 4; ++g) {
                    uint32_t word = 0;          // four codes: two bytes of nibbles, or four bytes
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        word |= (code_of(c * MM + 4 * g + i) & ((1u << CB) - 1)) << (CB * i);
                    }
                    const size_t pos = first + (size_t)(lane + 64 * c) * MM + 4 * g;      // position of the first of the four codes
                    if constexpr (CB == 4) *reinterpret_cast<uint16_t *>(out + pos / 2) = (uint16_t)word;
                    else *reinterpret_cast<uint32_t *>(out + pos) = word;
                }
        }
    }
    if constexpr (MODE == gen::kColAbsMax) {
        if (wave < rows) {
            // non-negative floats order like their bit patterns
#pragma unroll
            for (int r = 0; r < R; ++r)
                atomicMax(&col_absmax_bits[first + (lane + 64 * (r / MM)) * MM + (r % MM)], __float_as_uint(colmax[r]));
        }
    }
}


// K = N2 * MM for the sizes this file instantiates
bool general_size_supported(int K)
{
    switch (K) {
        case 768: case 1536: case 3072: case 6144: case 1280: case 2560: case 5120: case 1792: case 3584: return true;
        default: return false;
    }
}

template <int N2, int MM>
static hipError_t launch_general(const void *X, bool f32, int rows, const int8_t *signs, const float *mul, int mul_mode,
                                 uint8_t *packed, float *scale, unsigned int *colmax, const float *step, int step_stride,
                                 int bits, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    constexpr int ROWS = 4 / gen::waves_per_row(N2, MM);            // rows a block has in work
    int blocks = (rows + ROWS - 1) / ROWS;
    if (blocks > 256 * 8) blocks = 256 * 8;
    if (colmax != nullptr) blocks = std::max(1, std::min((rows + 8 * ROWS - 1) / (8 * ROWS), 256 * 2));   // eight rows or more per wave for the statistic
    const float qmax = (float)((1 << (code_width(bits) - 1)) - 1);
#define QVGGT_GEN(F32_, MODE_, CB_) \
    rotate_rows_general_kernel<N2, MM, F32_, MODE_, CB_><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, qmax)
    if (colmax != nullptr) {
        if (f32) QVGGT_GEN(true, gen::kColAbsMax, 4); else QVGGT_GEN(false, gen::kColAbsMax, 4);
    } else if (bits == 4) {
        if (f32) QVGGT_GEN(true, gen::kQuantize, 4); else QVGGT_GEN(false, gen::kQuantize, 4);
    } else {
        if (f32) QVGGT_GEN(true, gen::kQuantize, 8); else QVGGT_GEN(false, gen::kQuantize, 8);
    }
#undef QVGGT_GEN
    return hipGetLastError();
}

// colmax != nullptr: column absmax statistic (packed, scale unused); otherwise quantize with `bits`
hipError_t run_rotate_rows_general(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul, int mul_mode,
                                   uint8_t *packed, float *scale, unsigned int *colmax, const float *step, int step_stride,
                                   int bits, hipStream_t stream)
{
#define QVGGT_CASE(KK, N2, MM) \
    case KK: return launch_general<N2, MM>(X, f32, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, bits, stream);
    switch (K) {
        QVGGT_CASE(768, 64, 12)
        QVGGT_CASE(1536, 128, 12)
        QVGGT_CASE(3072, 256, 12)
        QVGGT_CASE(6144, 512, 12)
        QVGGT_CASE(1280, 64, 20)
        QVGGT_CASE(2560, 128, 20)
        QVGGT_CASE(5120, 256, 20)
        QVGGT_CASE(1792, 64, 28)
        QVGGT_CASE(3584, 128, 28)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_CASE
}

template <int N2, int MM>
static hipError_t launch_general_e2m3(const void *X, bool f32, int rows, const int8_t *signs, const float *mul, int mul_mode, uint8_t *out, float *scale,
                                      uint8_t *rows_out, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    const int group = gen::waves_per_row(N2, MM) > 1 && rows <= kFewSharedRows ? 1 : kE2m3Group;
    const int blocks = std::min((rows + group - 1) / group, 256 * 8);
    auto launch = [&](auto kernel) {
        kernel<<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, out, scale, nullptr, nullptr, 0, 7.0f, rows_out);
        return hipGetLastError();
    };
    if (rows_out != nullptr) return launch(f32 ? rotate_rows_general_kernel<N2, MM, true, gen::kQuantize, 6, true> : rotate_rows_general_kernel<N2, MM, false, gen::kQuantize, 6, true>);
    if (f32) return launch(rotate_rows_general_kernel<N2, MM, true, gen::kQuantize, 6>);
    if constexpr (paley_size(N2 * MM)) return hipErrorInvalidValue;               // bf16 activations: rotate_quant_paley.hip
    else return launch(rotate_rows_general_kernel<N2, MM, false, gen::kQuantize, 6>);
}

// the same rows as E2M3 blocks (dynamic 4-bit codes); rows_out: as packed rows too, or nullptr
hipError_t run_rotate_rows_general_e2m3(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul, int mul_mode, uint8_t *out,
                                        float *scale, uint8_t *rows_out, hipStream_t stream)
{
#define QVGGT_CASE(KK, N2, MM) \
    case KK: return launch_general_e2m3<N2, MM>(X, f32, rows, signs, mul, mul_mode, out, scale, rows_out, stream);
    switch (K) {
        QVGGT_CASE(768, 64, 12)
        QVGGT_CASE(1536, 128, 12)
        QVGGT_CASE(3072, 256, 12)
        QVGGT_CASE(6144, 512, 12)
        QVGGT_CASE(1280, 64, 20)
        QVGGT_CASE(2560, 128, 20)
        QVGGT_CASE(5120, 256, 20)
        QVGGT_CASE(1792, 64, 28)
        QVGGT_CASE(3584, 128, 28)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_CASE
}

}  // namespace qvggt
