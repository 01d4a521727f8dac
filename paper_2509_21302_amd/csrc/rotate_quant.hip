// Online kernel 1 and its offline twins: randomised Walsh-Hadamard rotation of rows,
// per-channel multiply, then either per-row quantization (activations per token, weights
// per output channel; 4-bit codes packed two per byte, or wider codes as int8) or a
// per-channel absmax (smoothing statistics).
//
// One wavefront owns one row at a time.  A row of K values lives in K/64 registers per
// lane; element e = c*(64*V) + lane*V + i sits in register c*V + i, where V = min(8, K/64)
// is the run a lane loads contiguously (16 bytes of bf16 when V = 8, so a wave reads 1 KiB
// per load instruction).  The transform is one butterfly per index bit (the Hadamard matrix
// is a Kronecker power of H_2, paper Sec. 3.2): bits inside i and c are register-to-register,
// the six lane bits go through cross-lane exchanges.
#include "paley.h"
#include "qvggt_common.h"
#include "rotate_rows.h"

namespace qvggt {

enum RowMode { kQuantize = 0, kColAbsMax = 1 };

// mul_mode 0: mul[j] used as given (inv_smooth, or 1/sqrt(K) when mul == nullptr)
// mul_mode 1: 1 / (K * mul[j])   (weights: c_j / sqrt(K) recovered from inv_smooth)
// CB: bits a stored code occupies (4: two per byte; 8: one int8 each; 6: 4-bit codes as E2M3 blocks, dynamic steps).  qmax: largest code, 2^(bits-1) - 1.
// LN: a LayerNorm of the row precedes everything else (quantize mode, K <= 4096: beyond that the row no longer fits the registers)
// ASYM: affine 4-bit codes over the row's range [min(0, min z), max(0, max z)], zero point to zero[row], nibbles hold u - 8
// BOTH (CB = 6): the codes also go out as rows of packed nibbles, to rows_out (the two forms a layer keeps)
template <int K, bool F32, int MODE, int CB, bool LN = false, bool ASYM = false, bool BOTH = false>
__global__ __launch_bounds__(256) void rotate_rows_kernel(const void *__restrict__ X, int rows,
                                                          const int8_t *__restrict__ signs,
                                                          const float *__restrict__ mul, int mul_mode,
                                                          uint8_t *__restrict__ packed,
                                                          float *__restrict__ scale,
                                                          unsigned int *__restrict__ col_absmax_bits,
                                                          const float *__restrict__ step, int step_stride, float qmax,
                                                          LnParams ln, float *__restrict__ zero = nullptr, uint8_t *__restrict__ rows_out = nullptr)
{
    // waves per row: one, or the four of a block where a row would take 128 registers of a lane (two copies of it with the multipliers:
    // one wave per SIMD).  A wave then has K / 4 consecutive elements, and two butterflies go over the wave number.
    // 34350 x 8192 bf16: 594 us with one wave per row.
    constexpr int WPR = K > 4096 ? 4 : 1, KW = K / WPR;
    constexpr int V = RowMap<KW>::V, C = RowMap<KW>::C, R = RowMap<KW>::R;
    constexpr bool kPermuted = (K == 1024 || K == 2048 || K == 4096) && MODE == kQuantize;
    constexpr bool E2M3 = (CB == 6);
    static_assert(!E2M3 || (MODE == kQuantize && !LN && !ASYM), "E2M3 blocks: dynamic 4-bit codes");
    static_assert(!BOTH || E2M3, "two forms of a layer's weight codes");
    __shared__ __attribute__((aligned(16))) uint8_t lds_stage[E2M3 ? E2m3Stage<K>::BYTES : kPermuted ? 4 * K : 16];
    const int lane = threadIdx.x & 63;
    const int sub = WPR > 1 ? (int)(threadIdx.x >> 6) : 0, first = sub * KW;       // this wave's part of a row
    const int group = !E2M3 || WPR == 1 || rows > kFewSharedRows ? kE2m3Group : 1;       // rows that leave together
    const int wave = WPR > 1 ? (int)blockIdx.x * (E2M3 ? group : 1) : (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int nwaves = WPR > 1 ? (int)gridDim.x : (int)gridDim.x * 4;
    __shared__ float4 exchange[WPR > 1 ? K / 4 : 1];
    __shared__ float red[2][4];

    // per-lane constants: signs (a mask per register while there is room, one bit otherwise) and channel multipliers
    constexpr bool SIGN_MASKS = R <= 32;
    uint32_t neg[SIGN_MASKS ? R : (R + 31) / 32];
#pragma unroll
    for (int w = 0; w < (SIGN_MASKS ? R : (R + 31) / 32); ++w) neg[w] = 0;
    // the normalisation at K = 4096 leaves no registers for the multipliers: read again for every row there
    constexpr bool KEEP_MUL = !(LN && R >= 64);
    float cm[KEEP_MUL ? R : 1];
    const float rs = 1.0f / sqrtf((float)K);
    // loads first (all in flight together), arithmetic afterwards: the set-up is one memory round trip, not one per element
    if (signs != nullptr) {
        int8_t sb[R];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int i = 0; i < V; ++i) sb[c * V + i] = signs[first + c * 64 * V + lane * V + i];
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (sb[r] < 0) neg[SIGN_MASKS ? r : r >> 5] |= SIGN_MASKS ? 0x80000000u : 1u << (r & 31);
    }
    if (!KEEP_MUL) {
    } else if (mul != nullptr) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int i = 0; i < V; ++i) cm[c * V + i] = mul[first + c * 64 * V + lane * V + i];
        if (mul_mode) {
#pragma unroll
            for (int r = 0; r < R; ++r) cm[r] = 1.0f / ((float)K * cm[r]);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) cm[r] = rs;
    }

    float colmax[MODE == kColAbsMax ? R : 1];
#pragma unroll
    for (int r = 0; r < (MODE == kColAbsMax ? R : 1); ++r) colmax[r] = 0.0f;
    // E2M3: a block takes a group of consecutive rows at a time, one per wave or (WPR > 1) one after the other; past the end: the last row, not
    // written
    const int last = group - 1;
    for (int row = wave; (E2M3 ? row & ~last : row) < rows; row += !(E2M3 && WPR > 1) ? nwaves : (row & last) == last ? group * nwaves - last : 1) {
        float x[R];
        load_row<KW, F32>(X, (size_t)(E2M3 ? min(row, rows - 1) : row) * WPR + sub, lane, x);
        if constexpr (LN) {
            static_assert(!LN || WPR == 1, "the normalisation sums over one wave");
            // LayerNorm of the token in fp32 (two passes over the registers), result rounded to the input's type as a separate
            // normalisation kernel would hand it on; gamma and beta come through the caches, this is the general path
            float s1 = 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) s1 += x[r];
            const float mean = sum_over_64_lanes(s1) * (1.0f / (float)K);
            float s2 = 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) { x[r] -= mean; s2 = fmaf(x[r], x[r], s2); }
            const float rstd = 1.0f / sqrtf(sum_over_64_lanes(s2) * (1.0f / (float)K) + ln.eps);
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int e = c * 64 * V + lane * V + i, r = c * V + i;
                    float y = x[r] * rstd;
                    const float gm = ln.gamma ? ln.gamma[e] : 1.0f, bt = ln.beta ? ln.beta[e] : 0.0f;
                    y = fmaf(y, gm, bt);
                    if constexpr (!F32) y = bf16_bits_to_float(pack_bf16x2(y, 0.0f) & 0xFFFFu);
                    x[r] = y;
                }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            x[r] = __uint_as_float(__float_as_uint(x[r]) ^ (SIGN_MASKS ? neg[r] : (neg[r >> 5] << (31 - (r & 31))) & 0x80000000u));
        fwht_row<KW>(x, lane);
        if constexpr (WPR > 1) wave_butterflies(x, exchange, sub, lane);
        const float *row_mul = mul;
        if constexpr (!KEEP_MUL) asm volatile("" : "+s"(row_mul));       // keeps the reads inside the loop
        auto multiplier = [&](int r) -> float {
            if constexpr (KEEP_MUL) {
                return cm[r];
            } else {
                const float m = row_mul != nullptr ? row_mul[first + (r / V) * 64 * V + lane * V + r % V] : rs;
                return (mul_mode && row_mul != nullptr) ? 1.0f / ((float)K * m) : m;
            }
        };
        float amax = 0.0f, nmin = 0.0f;       // ASYM: max(0, max z) and -min(0, min z)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[r] *= multiplier(r);
            if constexpr (ASYM) { amax = fmaxf(amax, x[r]); nmin = fmaxf(nmin, -x[r]); }
            else amax = fmaxf(amax, fabsf(x[r]));
        }

        if constexpr (MODE == kColAbsMax) {
            // the wave keeps a running maximum over its rows; one atomic per column after the loop
#pragma unroll
            for (int r = 0; r < R; ++r) colmax[r] = fmaxf(colmax[r], fabsf(x[r]));
        } else {
            // dynamic: the step comes from the row's absmax; static: it is given (per token or one for the tensor)
            float inv, delta, off = 0.0f;
            if constexpr (ASYM) {
                float hi = max_over_64_lanes(amax), nlo = max_over_64_lanes(nmin);
                if constexpr (WPR > 1) { hi = max_over_4_waves(hi, red[0]); nlo = max_over_4_waves(nlo, red[1]); }
                const float range = hi + nlo;
                const bool live = range >= 15.0f * kMinStep;
                delta = live ? range / 15.0f : 0.0f;
                inv = live ? 15.0f / range : 0.0f;
                const float zp = __builtin_rintf(nlo * inv);                  // rne(-lo / step), in [0, 15]
                off = zp - 8.0f;
                if (lane == 0 && sub == 0) zero[row] = zp;
            } else if (step != nullptr) {
                delta = step[(size_t)row * step_stride];
                inv = delta >= kMinStep ? 1.0f / delta : 0.0f;
            } else {
                amax = max_over_64_lanes(amax);
                if constexpr (WPR > 1) amax = max_over_4_waves(amax, red[0]);
                const bool live = amax >= qmax * kMinStep;
                delta = live ? amax / qmax : 0.0f;
                inv = live ? qmax / amax : 0.0f;
            }
            if (lane == 0 && sub == 0 && (!E2M3 || row < rows)) scale[row] = delta;
            const int q_hi = (int)qmax, q_lo = -q_hi - 1;
            // a step from the row's own maximum bounds |x * inv| by qmax (1 + 2^-22): rounding cannot leave the range, and the code is the low
            // bits of one fma.  (inv is 0 for a row without a step, or whose values overflowed: the general form gives codes 0 there.)
            const bool bounded = !ASYM && step == nullptr && inv > 0.0f;
            auto code_of = [&](int r) -> uint32_t {       // two's complement in the low CB bits, anything above
                if (bounded) return __float_as_uint(fmaf(x[r], inv, kRoundMagic));
                const int q = (int)__builtin_rintf(ASYM ? fmaf(x[r], inv, off) : x[r] * inv);
                return (uint32_t)min(q_hi, max(q_lo, q));
            };
            if constexpr (E2M3) {
                uint8_t *stage = lds_stage + (row & last) * E2m3Stage<K>::PITCH;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int e0 = first + c * 64 * V + lane * V;
                    if constexpr (kPermuted || V < 4) {
#pragma unroll
                        for (int i = 0; i < V; ++i) stage[code_position(e0 + i, K)] = (uint8_t)code_of(c * V + i);
                    } else {
#pragma unroll
                        for (int i = 0; i < V; i += 4)
                            *reinterpret_cast<uint32_t *>(stage + e0 + i) = low_bytes(code_of(c * V + i), code_of(c * V + i + 1), code_of(c * V + i + 2), code_of(c * V + i + 3));
                    }
                }
                if (WPR == 1 || (row & last) == last) {       // the same for the whole block
                    __syncthreads();
                    flush_e2m3<K, BOTH>(lds_stage, row & ~last, group, rows, packed, rows_out);
                    __syncthreads();
                }
                continue;
            }
            uint8_t *out = packed + (size_t)row * (K * CB / 8);
            if constexpr (K == 1024 || K == 2048 || K == 4096) {
                // permuted layout: scatter the codes as bytes into the wave's LDS row at their positions,
                // then every lane packs K/64 consecutive positions
                uint8_t *stage = lds_stage + (threadIdx.x >> 6) * K;
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int i = 0; i < V; ++i) stage[code_position(c * 64 * V + lane * V + i, K)] = (uint8_t)code_of(c * V + i);
                lanes_exchange_fence();
                constexpr int PER_LANE = K / 64;      // positions per lane, a multiple of 16
                if constexpr (CB == 8) {
#pragma unroll
                    for (int b = 0; b < PER_LANE / 16; ++b)
                        *reinterpret_cast<uint4 *>(out + lane * PER_LANE + 16 * b) = *reinterpret_cast<const uint4 *>(stage + lane * PER_LANE + 16 * b);
                } else {
#pragma unroll
                    for (int b = 0; b < PER_LANE / 8; ++b) {
                        const uint2 v = *reinterpret_cast<const uint2 *>(stage + lane * PER_LANE + 8 * b);
                        // bytes hold one code each (low nibble): squeeze 8 bytes into 8 nibbles
                        uint32_t lo = v.x & 0x0F0F0F0Fu, hi = v.y & 0x0F0F0F0Fu;
                        lo = (lo | (lo >> 4)) & 0x00FF00FFu; lo = (lo | (lo >> 8)) & 0x0000FFFFu;
                        hi = (hi | (hi >> 4)) & 0x00FF00FFu; hi = (hi | (hi >> 8)) & 0x0000FFFFu;
                        *reinterpret_cast<uint32_t *>(out + lane * (PER_LANE / 2) + 4 * b) = lo | (hi << 16);
                    }
                }
                lanes_exchange_fence();
            } else {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                uint64_t word = 0;
#pragma unroll
                for (int i = 0; i < V; ++i) word |= (uint64_t)(code_of(c * V + i) & ((1u << CB) - 1)) << (CB * i);
                // natural order: element e -> code slot e; a lane's V codes are V * CB / 8 consecutive bytes
                const int byte0 = (first + c * 64 * V + lane * V) * CB / 8;
                if constexpr (V * CB == 64) *reinterpret_cast<uint2 *>(out + byte0) = make_uint2((uint32_t)word, (uint32_t)(word >> 32));
                else if constexpr (V * CB == 32) *reinterpret_cast<uint32_t *>(out + byte0) = (uint32_t)word;
                else if constexpr (V * CB == 16) *reinterpret_cast<uint16_t *>(out + byte0) = (uint16_t)word;
                else out[byte0] = (uint8_t)word;
            }
            }
        }
    }
    if constexpr (MODE == kColAbsMax) {
        if (wave < rows) {
            // non-negative floats order like their bit patterns
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int i = 0; i < V; ++i)
                    atomicMax(&col_absmax_bits[first + c * 64 * V + lane * V + i], __float_as_uint(colmax[c * V + i]));
        }
    }
}

// ---------------------------------------------------------------------------------------
// small helpers of the offline path

__global__ void fill_u32_kernel(unsigned int *p, int n, unsigned int v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// in place: buf[j] holds w_j = max_o |W H|[o, j] on entry, inv_smooth[j] = 1 / (sqrt(K) c_j) on exit
__global__ void smooth_factor_kernel(float *buf, const float *__restrict__ act_absmax, int K, float alpha)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= K) return;
    const float floor_ = 1e-5f;
    float a = fmaxf(act_absmax[j], floor_), w = fmaxf(buf[j], floor_);
    float c = powf(a, alpha) / powf(w, 1.0f - alpha);
    buf[j] = 1.0f / (sqrtf((float)K) * c);
}

// a given smoothing factor c[j] -> inv_smooth[j] = 1 / (sqrt(K) c_j)
__global__ void inv_from_factor_kernel(float *buf, const float *__restrict__ c, int K)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < K) buf[j] = 1.0f / (sqrtf((float)K) * c[j]);
}

__global__ void fill_f32_kernel(float *p, int n, float v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// int8 codes in natural order <-> packed rows in the library layout
__global__ void pack_int4_kernel(const int8_t *__restrict__ codes, size_t rows, int K, uint8_t *__restrict__ packed)
{
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one output byte each
    if (idx >= rows * (size_t)(K / 2)) return;
    size_t row = idx / (K / 2);
    int byte = (int)(idx % (K / 2));
    int e0 = code_element(2 * byte, K), e1 = code_element(2 * byte + 1, K);
    uint8_t lo = (uint8_t)codes[row * K + e0] & 0xF, hi = (uint8_t)codes[row * K + e1] & 0xF;
    packed[idx] = lo | (hi << 4);
}

__global__ void unpack_int4_kernel(const uint8_t *__restrict__ packed, size_t rows, int K, int8_t *__restrict__ codes)
{
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one natural element each
    if (idx >= rows * (size_t)K) return;
    size_t row = idx / K;
    int e = (int)(idx % K);
    int p = code_position(e, K);
    uint8_t b = packed[row * (K / 2) + p / 2];
    int nib = (p & 1) ? (b >> 4) : (b & 0xF);
    codes[idx] = (int8_t)(nib >= 8 ? nib - 16 : nib);
}

// int8 codes: natural order <-> the library's position order (the same map as for packed rows, one byte per position)
// sums[o] = sum_j code[o, j] over a row of packed 4-bit codes (any position order): one wave per row
__global__ __launch_bounds__(256) void code_sums_kernel(const uint8_t *__restrict__ packed, int rows, int K, float *__restrict__ sums)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const uint32_t *p = reinterpret_cast<const uint32_t *>(packed + (size_t)row * (K / 2));
    int s = 0;
    for (int i = lane; i < K / 8; i += 64) {
        const uint32_t v = p[i];
#pragma unroll
        for (int n = 0; n < 8; ++n) s += (int)(v << (28 - 4 * n)) >> 28;      // sign-extended nibble n
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m);
    if (lane == 0) sums[row] = (float)s;                                        // |s| <= 8 K: exact
}

__global__ void layout_int8_kernel(const int8_t *__restrict__ src, size_t rows, int K, int8_t *__restrict__ dst, int to_library)
{
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one output byte each
    if (idx >= rows * (size_t)K) return;
    size_t row = idx / K;
    int o = (int)(idx % K);
    dst[idx] = src[row * K + (to_library ? code_element(o, K) : code_position(o, K))];
}

// ---------------------------------------------------------------------------------------
// host-side launchers (called from api.hip)

// sizes 2^n * m (m = 12, 20, 28): rotate_quant_general.hip
bool general_size_supported(int K);
hipError_t run_rotate_rows_general(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul, int mul_mode,
                                   uint8_t *packed, float *scale, unsigned int *colmax, const float *step, int step_stride,
                                   int bits, hipStream_t stream);

hipError_t run_rotate_rows_general_e2m3(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul, int mul_mode, uint8_t *out,
                                        float *scale, uint8_t *rows_out, hipStream_t stream);
hipError_t run_rotate_quant_paley(const void *X, int rows, int K, const int8_t *signs, const float *mul, uint8_t *out, float *scale,
                                  const float *step, int step_stride, int form, float qmax, hipStream_t stream);
// Activation rows (mul_mode 0) with a Paley factor, or of 8192 values, whatever their number: the general kernel sums in another order, and a row's codes do not
// depend on how many rows come with it.  fp32 values are no exact operands of the matrix instruction; weights keep the codes they have had.
static bool paley_on_matrix_cores(bool f32, int K, int mul_mode) { return !f32 && mul_mode == 0 && paley_size(K); }

// rows_out (CB = 6): the packed rows, or nullptr
template <int MODE, int CB>
static hipError_t launch_rotate_rows(const void *X, bool f32, int rows, int K, const int8_t *signs,
                                     const float *mul, int mul_mode, uint8_t *packed, float *scale,
                                     unsigned int *colmax, const float *step, int step_stride, float qmax, hipStream_t stream,
                                     uint8_t *rows_out = nullptr)
{
    if (rows <= 0) return hipSuccess;
    const int waves_per_block = 4;
    // four waves share a row beyond 4096 values; E2M3 blocks leave in groups of rows
    const int rows_per_block = K > 4096 && (CB != 6 || rows <= kFewSharedRows) ? 1 : waves_per_block;
    int blocks = (rows + rows_per_block - 1) / rows_per_block;
    // up to eight blocks per compute unit; the column statistic takes fewer waves for small inputs so that each folds several
    // rows into its running maximum before touching the shared result
    const int max_blocks = (MODE == kColAbsMax) ? 256 * 2 : 256 * 8;
    if (MODE == kColAbsMax) blocks = (rows + 8 * rows_per_block - 1) / (8 * rows_per_block);     // eight rows or more per wave: the atomics at the end are what costs
    if (blocks > max_blocks) blocks = max_blocks;
    if (blocks < 1) blocks = 1;
#define QVGGT_LAUNCH(KK)                                                                                     \
    case KK:                                                                                                 \
        if (f32) rotate_rows_kernel<KK, true, MODE, CB><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, qmax, LnParams{nullptr, nullptr, 0.0f, 0}); \
        else if constexpr (CB == 6 && paley_size(KK)) return hipErrorInvalidValue;      /* bf16 activations: rotate_quant_paley.hip */     \
        else rotate_rows_kernel<KK, false, MODE, CB><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, qmax, LnParams{nullptr, nullptr, 0.0f, 0});    \
        break;
    if constexpr (CB == 6) {
        if (rows_out != nullptr) {
#define QVGGT_LAUNCH_BOTH(KK)                                                                                \
    case KK:                                                                                                 \
        if (f32) rotate_rows_kernel<KK, true, MODE, CB, false, false, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, qmax, LnParams{nullptr, nullptr, 0.0f, 0}, nullptr, rows_out); \
        else rotate_rows_kernel<KK, false, MODE, CB, false, false, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, mul_mode, packed, scale, colmax, step, step_stride, qmax, LnParams{nullptr, nullptr, 0.0f, 0}, nullptr, rows_out);    \
        return hipGetLastError();
            switch (K) {
                QVGGT_LAUNCH_BOTH(128)
                QVGGT_LAUNCH_BOTH(256)
                QVGGT_LAUNCH_BOTH(512)
                QVGGT_LAUNCH_BOTH(8192)
                default: return hipErrorInvalidValue;
            }
#undef QVGGT_LAUNCH_BOTH
        }
    }
    switch (K) {
        QVGGT_LAUNCH(128)
        QVGGT_LAUNCH(256)
        QVGGT_LAUNCH(512)
        QVGGT_LAUNCH(1024)
        QVGGT_LAUNCH(2048)
        QVGGT_LAUNCH(4096)
        QVGGT_LAUNCH(8192)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_LAUNCH
    return hipGetLastError();
}

hipError_t run_rotate_quant_mfma(const void *X, int rows, int K, const int8_t *signs, const float *mul, int mul_mode,
                                 uint8_t *packed, float *scale, const float *step, int step_stride, int bits,
                                 hipStream_t stream);
hipError_t run_rotated_col_absmax_mfma(const void *X, int rows, int K, const int8_t *signs, unsigned int *absmax_bits,
                                       hipStream_t stream);

// bits: 4 (packed nibbles) or 5..8 (int8 codes in [-2^(bits-1), 2^(bits-1) - 1])
hipError_t run_rotate_smooth_quant(const void *X, bool f32, int rows, int K, const int8_t *signs,
                                   const float *mul, int mul_mode, uint8_t *packed, float *scale,
                                   const float *step, int step_stride, int bits, hipStream_t stream)
{
    const float qmax = (float)((1 << (code_width(bits) - 1)) - 1);
    if (paley_on_matrix_cores(f32, K, mul_mode))
        return run_rotate_quant_paley(X, rows, K, signs, mul, packed, scale, step, step_stride, bits == 4 ? 4 : 8, qmax, stream);
    if (general_size_supported(K))
        return run_rotate_rows_general(X, f32, rows, K, signs, mul, mul_mode, packed, scale, nullptr, step, step_stride, bits, stream);
    // bf16 rows of the sizes VGGT-1B uses go to the matrix-core kernel; everything else to the generic one
    if (!f32 && (K == 1024 || K == 2048 || K == 4096))
        return run_rotate_quant_mfma(X, rows, K, signs, mul, mul_mode, packed, scale, step, step_stride, bits, stream);
    if (bits == 4)
        return launch_rotate_rows<kQuantize, 4>(X, f32, rows, K, signs, mul, mul_mode, packed, scale, nullptr, step, step_stride, qmax, stream);
    return launch_rotate_rows<kQuantize, 8>(X, f32, rows, K, signs, mul, mul_mode, packed, scale, nullptr, step, step_stride, qmax, stream);
}

// rotation + smoothing + per-row 4-bit codes as E2M3 blocks for the rows that the matrix-core kernel does not take: f32, or other sizes.
// rows_out: the same codes as packed rows, or nullptr (K other than 1024, 2048 and 4096)
hipError_t run_rotate_rows_e2m3(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul, int mul_mode, uint8_t *out,
                                float *scale, uint8_t *rows_out, hipStream_t stream)
{
    if (rows_out == nullptr && paley_on_matrix_cores(f32, K, mul_mode))
        return run_rotate_quant_paley(X, rows, K, signs, mul, out, scale, nullptr, 0, 6, 7.0f, stream);
    if (general_size_supported(K)) return run_rotate_rows_general_e2m3(X, f32, rows, K, signs, mul, mul_mode, out, scale, rows_out, stream);
    return launch_rotate_rows<kQuantize, 6>(X, f32, rows, K, signs, mul, mul_mode, out, scale, nullptr, nullptr, 0, 7.0f, stream, rows_out);
}

hipError_t run_ln_rotate_quant_mfma(const void *X, int rows, const int8_t *signs, const float *mul, uint8_t *packed, float *scale,
                                    LnParams ln, hipStream_t stream);

// LayerNorm + rotation + smoothing + per-token 4-bit quantization in one kernel (power-of-two K)
hipError_t run_ln_rotate_smooth_quant(const void *X, bool f32, int rows, int K, LnParams ln, const int8_t *signs, const float *mul,
                                      uint8_t *packed, float *scale, hipStream_t stream)
{
    if (!f32 && K == 1024) return run_ln_rotate_quant_mfma(X, rows, signs, mul, packed, scale, ln, stream);
    if (rows <= 0) return hipSuccess;
    int blocks = (rows + 3) / 4;
    if (blocks > 256 * 8) blocks = 256 * 8;
#define QVGGT_LAUNCH_LN(KK)                                                                                                            \
    case KK:                                                                                                                           \
        if (f32) rotate_rows_kernel<KK, true, kQuantize, 4, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, 0, packed, scale, nullptr, nullptr, 0, 7.0f, ln); \
        else rotate_rows_kernel<KK, false, kQuantize, 4, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, 0, packed, scale, nullptr, nullptr, 0, 7.0f, ln);    \
        break;
    switch (K) {
        QVGGT_LAUNCH_LN(128)
        QVGGT_LAUNCH_LN(256)
        QVGGT_LAUNCH_LN(512)
        QVGGT_LAUNCH_LN(1024)
        QVGGT_LAUNCH_LN(2048)
        QVGGT_LAUNCH_LN(4096)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_LAUNCH_LN
    return hipGetLastError();
}

hipError_t run_rotate_quant_asym_mfma(const void *X, int rows, int K, const int8_t *signs, const float *mul, uint8_t *packed,
                                      float *scale, float *zero, hipStream_t stream);

// rotation + smoothing + per-token affine 4-bit codes with zero points (power-of-two K)
hipError_t run_rotate_smooth_quant_asym(const void *X, bool f32, int rows, int K, const int8_t *signs, const float *mul,
                                        uint8_t *packed, float *scale, float *zero, hipStream_t stream)
{
    if (!f32 && (K == 1024 || K == 2048 || K == 4096))
        return run_rotate_quant_asym_mfma(X, rows, K, signs, mul, packed, scale, zero, stream);
    if (rows <= 0) return hipSuccess;
    int blocks = K > 4096 ? rows : (rows + 3) / 4;
    if (blocks > 256 * 8) blocks = 256 * 8;
    const LnParams no_ln{nullptr, nullptr, 0.0f, 0};
#define QVGGT_LAUNCH_ASYM(KK)                                                                                                          \
    case KK:                                                                                                                           \
        if (f32) rotate_rows_kernel<KK, true, kQuantize, 4, false, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, 0, packed, scale, nullptr, nullptr, 0, 7.0f, no_ln, zero); \
        else rotate_rows_kernel<KK, false, kQuantize, 4, false, true><<<blocks, 256, 0, stream>>>(X, rows, signs, mul, 0, packed, scale, nullptr, nullptr, 0, 7.0f, no_ln, zero);    \
        break;
    switch (K) {
        QVGGT_LAUNCH_ASYM(128)
        QVGGT_LAUNCH_ASYM(256)
        QVGGT_LAUNCH_ASYM(512)
        QVGGT_LAUNCH_ASYM(1024)
        QVGGT_LAUNCH_ASYM(2048)
        QVGGT_LAUNCH_ASYM(4096)
        QVGGT_LAUNCH_ASYM(8192)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_LAUNCH_ASYM
    return hipGetLastError();
}

hipError_t run_rotated_col_absmax(const void *X, bool f32, int rows, int K, const int8_t *signs,
                                  float *absmax, hipStream_t stream)
{
    fill_u32_kernel<<<(K + 255) / 256, 256, 0, stream>>>(reinterpret_cast<unsigned int *>(absmax), K, 0u);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!f32 && (K == 1024 || K == 2048 || K == 4096))
        return run_rotated_col_absmax_mfma(X, rows, K, signs, reinterpret_cast<unsigned int *>(absmax), stream);
    if (general_size_supported(K))
        return run_rotate_rows_general(X, f32, rows, K, signs, nullptr, 0, nullptr, nullptr, reinterpret_cast<unsigned int *>(absmax),
                                       nullptr, 0, 4, stream);
    return launch_rotate_rows<kColAbsMax, 4>(X, f32, rows, K, signs, nullptr, 0, nullptr, nullptr,
                                             reinterpret_cast<unsigned int *>(absmax), nullptr, 0, 7.0f, stream);
}

hipError_t run_smooth_factor(float *buf, const float *act_absmax, int K, float alpha, hipStream_t stream)
{
    smooth_factor_kernel<<<(K + 255) / 256, 256, 0, stream>>>(buf, act_absmax, K, alpha);
    return hipGetLastError();
}

hipError_t run_inv_from_factor(float *buf, const float *c, int K, hipStream_t stream)
{
    inv_from_factor_kernel<<<(K + 255) / 256, 256, 0, stream>>>(buf, c, K);
    return hipGetLastError();
}

hipError_t run_fill_f32(float *p, int n, float v, hipStream_t stream)
{
    fill_f32_kernel<<<(n + 255) / 256, 256, 0, stream>>>(p, n, v);
    return hipGetLastError();
}

hipError_t run_pack_int4(const int8_t *codes, int rows, int K, uint8_t *packed, hipStream_t stream)
{
    size_t n = (size_t)rows * (K / 2);
    if (n == 0) return hipSuccess;
    pack_int4_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(codes, (size_t)rows, K, packed);
    return hipGetLastError();
}

hipError_t run_layout_int8(const int8_t *src, int rows, int K, int8_t *dst, int to_library, hipStream_t stream)
{
    size_t n = (size_t)rows * K;
    if (n == 0) return hipSuccess;
    layout_int8_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(src, (size_t)rows, K, dst, to_library);
    return hipGetLastError();
}

// int8 rows in library order [rows, K] -> int8 blocks (K-tiles of 64 bytes outermost inside 128-row blocks, chunks swizzled)
__global__ __launch_bounds__(256) void int8_to_blocks_kernel(const int8_t *__restrict__ src, size_t rows, int K, uint8_t *__restrict__ dst)
{
    const size_t chunks_per_row = (size_t)K / 16;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * chunks_per_row) return;
    const size_t row = idx / chunks_per_row;
    const int ch = (int)(idx - row * chunks_per_row), kt = ch >> 2, slot = (ch & 3) ^ (int)((row & 15) >> 2);
    const uint4 v = *reinterpret_cast<const uint4 *>(src + row * (size_t)K + (size_t)ch * 16);
    *reinterpret_cast<uint4 *>(dst + ((row / 128) * (size_t)(K / 64) + kt) * 8192 + (row % 128) * 64 + slot * 16) = v;
}

hipError_t run_int8_to_blocks(const int8_t *src, int rows, int K, uint8_t *dst, hipStream_t stream)
{
    const size_t n = (size_t)rows * (K / 16);
    if (n == 0) return hipSuccess;
    int8_to_blocks_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(src, (size_t)rows, K, dst);
    return hipGetLastError();
}

hipError_t run_code_sums(const uint8_t *packed, int rows, int K, float *sums, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    code_sums_kernel<<<(rows + 3) / 4, 256, 0, stream>>>(packed, rows, K, sums);
    return hipGetLastError();
}

hipError_t run_unpack_int4(const uint8_t *packed, int rows, int K, int8_t *codes, hipStream_t stream)
{
    size_t n = (size_t)rows * K;
    if (n == 0) return hipSuccess;
    unpack_int4_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(packed, (size_t)rows, K, codes);
    return hipGetLastError();
}

}  // namespace qvggt
