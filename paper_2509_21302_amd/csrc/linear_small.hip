// A whole packed 4-bit layer in one launch, for small calls: rotation, smoothing, codes, product and epilogue.
//
// A call of a few hundred rows or less is two launch-to-drain latencies and two launches' host work (3.6 us each); its arithmetic is nothing beside
// them.  Here a block takes BT tokens and 256 channels: its eight waves rotate and quantize the tokens (as rotate_rows_kernel does: one wave
// per row, the same operations on the same values), the codes meet in LDS as E2M3 numbers, and every wave multiplies them with its 32
// channels' weights, which it asked for before anything else.  The tokens are rotated again for every 256 channels: the price, and what the rule
// at the end of this file weighs.  Codes, steps, sums and Y are those of the two kernels, bit for bit.
#include "qvggt_common.h"
#include "rotate_rows.h"

#include <algorithm>

namespace qvggt {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int SM_WAVES = 8, SM_BN = SM_WAVES * 32;
constexpr int U_BYTES = 48, RB_BYTES = 128 * U_BYTES;        // the E2M3 operand format, see gemm_e2m3.hip

template <int K, int BT>
struct SmallCfg {
    static constexpr int UNITS = K / 64, CODE_PITCH = K + 64;
    static constexpr int X_BYTES = UNITS * 32 * U_BYTES;     // E2M3 codes [unit][32 rows][48 bytes]
    static constexpr int CODE_BYTES = BT * CODE_PITCH;       // the same codes as bytes, before
    static constexpr int EP_PITCH = 64 + 16, EP_BYTES = SM_WAVES * 32 * EP_PITCH;      // a wave's 32 x 32 results on their way to rows
};

template <int K, bool F32, int BT>
__global__ __launch_bounds__(SM_WAVES * 64) void linear_small_kernel(const void *__restrict__ X, int M, int N, const int8_t *__restrict__ signs,
                                                                     const float *__restrict__ mul, const uint8_t *__restrict__ Wf,
                                                                     const float *__restrict__ sw, const uint16_t *__restrict__ bias,
                                                                     uint16_t *__restrict__ Y, int tiles_n)
{
    using C = SmallCfg<K, BT>;
    constexpr int V = RowMap<K>::V, CH = RowMap<K>::C, R = RowMap<K>::R, ROWS = BT / SM_WAVES, UNITS = C::UNITS;
    static_assert(BT % SM_WAVES == 0 && BT <= 32, "a wave takes whole rows, a token sub-tile is 32");
    constexpr bool PERMUTED = K == 1024 || K == 2048 || K == 4096;
    __shared__ __attribute__((aligned(16))) uint8_t xf[C::X_BYTES];
    __shared__ __attribute__((aligned(16))) uint8_t scratch[C::CODE_BYTES > C::EP_BYTES ? C::CODE_BYTES : C::EP_BYTES];
    __shared__ float sx[32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tm = (int)blockIdx.x / tiles_n, tn = (int)blockIdx.x % tiles_n;
    const int row0 = tm * BT, col0 = tn * SM_BN + wave * 32;

    // ---- the wave's weights and its lanes' scales: 32 channels, all of K; past N: the last ones again (not written)
    const int frow = lane & 31, fhalf = lane >> 5;
    const int wcol = min(col0, (N - 1) & ~31);
    const uint8_t *wp = Wf + (size_t)(wcol / 128) * UNITS * RB_BYTES + (wcol % 128 + frow) * U_BYTES;
    v8i W[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const v4i lo = *reinterpret_cast<const v4i *>(wp + u * RB_BYTES + fhalf * 16);
        const int2 hi = *reinterpret_cast<const int2 *>(wp + u * RB_BYTES + 32 + fhalf * 8);
        W[u][0] = lo[0]; W[u][1] = lo[1]; W[u][2] = lo[2]; W[u][3] = lo[3]; W[u][4] = hi.x; W[u][5] = hi.y; W[u][6] = 0; W[u][7] = 0;
    }
    float4 swq[4];
    uint2 bq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {                            // channels 8 q + 4 fhalf .. + 3 of the wave's 32
        const int n = min(col0 + 8 * q + 4 * fhalf, N - 4);
        swq[q] = *reinterpret_cast<const float4 *>(sw + n);
        bq[q] = bias != nullptr ? *reinterpret_cast<const uint2 *>(bias + n) : make_uint2(0u, 0u);
    }

    // ---- kernel 1 on rows wave, wave + 8, ...; past M: the last row again (not written)
    float x[ROWS][R];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) load_row<K, F32>(X, (size_t)min(row0 + wave + SM_WAVES * i, M - 1), lane, x[i]);
    float cm[R];
    uint32_t neg[R];
    const float rs = 1.0f / sqrtf((float)K);
#pragma unroll
    for (int r = 0; r < R; ++r) { neg[r] = 0u; cm[r] = rs; }
    // a lane's V values of a chunk are consecutive: whole words, all loads in flight together
    if (signs != nullptr) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            int8_t sb[V];
            __builtin_memcpy(sb, __builtin_assume_aligned(signs + c * 64 * V + lane * V, V), V);
#pragma unroll
            for (int k = 0; k < V; ++k) neg[c * V + k] = ((uint32_t)(uint8_t)sb[k] & 0x80u) << 24;
        }
    }
    if (mul != nullptr) {
#pragma unroll
        for (int c = 0; c < CH; ++c) __builtin_memcpy(cm + c * V, __builtin_assume_aligned(mul + c * 64 * V + lane * V, V >= 4 ? 16 : 8), V * sizeof(float));
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int t = wave + SM_WAVES * i;
#pragma unroll
        for (int r = 0; r < R; ++r) x[i][r] = __uint_as_float(__float_as_uint(x[i][r]) ^ neg[r]);
        fwht_row<K>(x[i], lane);
        float amax = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) { x[i][r] *= cm[r]; amax = fmaxf(amax, fabsf(x[i][r])); }
        amax = max_over_64_lanes(amax);
        const float qmax = 7.0f;
        const bool live = amax >= qmax * kMinStep;
        const float inv = live ? qmax / amax : 0.0f;
        if (lane == 0) sx[t] = live ? amax / qmax : 0.0f;
        const bool bounded = inv > 0.0f;                     // as in rotate_rows_kernel
        auto code_of = [&](int r) -> uint32_t {
            if (bounded) return __float_as_uint(fmaf(x[i][r], inv, kRoundMagic));
            return (uint32_t)min(7, max(-8, (int)__builtin_rintf(x[i][r] * inv)));
        };
        uint8_t *codes = scratch + t * C::CODE_PITCH;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int e0 = c * 64 * V + lane * V;
            if constexpr (PERMUTED || V < 4) {
#pragma unroll
                for (int k = 0; k < V; ++k) codes[code_position(e0 + k, K)] = (uint8_t)code_of(c * V + k);
            } else {
#pragma unroll
                for (int k = 0; k < V; k += 4)
                    *reinterpret_cast<uint32_t *>(codes + e0 + k) = low_bytes(code_of(c * V + k), code_of(c * V + k + 1), code_of(c * V + k + 2), code_of(c * V + k + 3));
            }
        }
    }
    __syncthreads();
    for (int t = tid; t < BT * UNITS * 2; t += SM_WAVES * 64) {          // 32 codes each: unit, row, half
        const int h = t & 1, r = (t >> 1) % BT, unit = (t >> 1) / BT;
        const e2m3_v6u blob = e2m3_blob(scratch + r * C::CODE_PITCH + 64 * unit + 32 * h);
        uint8_t *u = xf + (unit * 32 + r) * U_BYTES;
        *reinterpret_cast<uint4 *>(u + h * 16) = make_uint4(blob[0], blob[1], blob[2], blob[3]);
        *reinterpret_cast<uint2 *>(u + 32 + h * 8) = make_uint2(blob[4], blob[5]);
    }
    __syncthreads();

    // ---- products: two chains of MFMAs (sums of integers: any order gives the same); rows past BT hold whatever is there
    v16f acc[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[s][r] = 0.0f;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const uint8_t *p = xf + (u * 32 + frow) * U_BYTES;
        const v4i lo = *reinterpret_cast<const v4i *>(p + fhalf * 16);
        const int2 hi = *reinterpret_cast<const int2 *>(p + 32 + fhalf * 8);
        v8i xv;
        xv[0] = lo[0]; xv[1] = lo[1]; xv[2] = lo[2]; xv[3] = lo[3]; xv[4] = hi.x; xv[5] = hi.y; xv[6] = 0; xv[7] = 0;
        acc[u & 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(W[u], xv, acc[u & 1], 2, 2, 0, 0, 0, 0);
    }

    // ---- epilogue: lane = token (lane % 32) and channels 8 q + 4 (lane / 32) .. + 3; rows through a wave-private tile (the code bytes are done with)
    uint8_t *ep = scratch + wave * (32 * C::EP_PITCH);
    const float st = sx[min(frow, BT - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float a[4] = {acc[0][4 * q] + acc[1][4 * q], acc[0][4 * q + 1] + acc[1][4 * q + 1], acc[0][4 * q + 2] + acc[1][4 * q + 2], acc[0][4 * q + 3] + acc[1][4 * q + 3]};
        const float y0 = fmaf(a[0], swq[q].x * st, __uint_as_float(bq[q].x << 16)), y1 = fmaf(a[1], swq[q].y * st, __uint_as_float(bq[q].x & 0xFFFF0000u));
        const float y2 = fmaf(a[2], swq[q].z * st, __uint_as_float(bq[q].y << 16)), y3 = fmaf(a[3], swq[q].w * st, __uint_as_float(bq[q].y & 0xFFFF0000u));
        *reinterpret_cast<uint2 *>(ep + frow * C::EP_PITCH + (8 * q + 4 * fhalf) * 2) = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
    }
    lanes_exchange_fence();
#pragma unroll
    for (int it = 0; it < (BT + 15) / 16; ++it) {            // 16 tokens of 64 bytes per store
        const int t = it * 16 + (lane >> 2), n = col0 + (lane & 3) * 8, m = row0 + t;
        const uint4 v = *reinterpret_cast<const uint4 *>(ep + t * C::EP_PITCH + (lane & 3) * 16);
        if (t < BT && m < M && n < N) *reinterpret_cast<uint4 *>(Y + (size_t)m * N + n) = v;
    }
}

}  // namespace

static int small_blocks(int M, int N, int rows) { return (M + rows - 1) / rows * ((N + SM_BN - 1) / SM_BN); }

// One block per compute unit, so that nothing waits for a block to end, and sizes whose rows a wave rotates in a few hundred instructions: the two
// kernels / this one, us a call, host and device together (M x K -> N): 16 x 128 -> 208 6.7 / 3.4, 2275 x 128 -> 464 8.6 / 5.3, 26 x 256 -> 144
// 6.6 / 4.0, 1454 x 256 -> 816 8.9 / 6.6, 22 x 512 -> 128 6.7 / 5.1, 312 x 512 -> 464 8.4 / 6.7.  Past a block per unit: 427 x 512 -> 2480 (270
// blocks) 8.9 / 9.1, 2857 x 512 -> 1392 11.2 / 21.  At K = 1024 (f32): 146 -> 208 7.7 / 10.0.
bool linear_small_pays(int M, int N, int K) { return (K == 128 || K == 256 || K == 512) && small_blocks(M, N, K == 512 ? 16 : 32) <= 256; }

hipError_t run_linear_small(const void *X, bool f32, int M, int N, int K, const int8_t *signs, const float *mul, const uint8_t *Wf, const float *sw,
                            const void *bias, void *Y, hipStream_t stream)
{
    if (M <= 0) return hipSuccess;
    const int tiles_n = (N + SM_BN - 1) / SM_BN;
    // eight tokens per block (one row per wave) or sixteen while that many blocks have a compute unit each
    const int rows = small_blocks(M, N, 8) <= 256 ? 8 : K == 512 || small_blocks(M, N, 16) <= 256 ? 16 : 32;
#define QVGGT_SMALL(KK, F32, BT)                                                                                                         \
    linear_small_kernel<KK, F32, BT><<<small_blocks(M, N, BT), SM_WAVES * 64, 0, stream>>>(X, M, N, signs, mul, Wf, sw, static_cast<const uint16_t *>(bias), static_cast<uint16_t *>(Y), tiles_n)
#define QVGGT_SMALL_ROWS(KK, BT)           \
    do {                                   \
        if (f32) QVGGT_SMALL(KK, true, BT); \
        else QVGGT_SMALL(KK, false, BT);   \
    } while (0)
    switch (K) {
        case 128: if (rows == 8) QVGGT_SMALL_ROWS(128, 8); else if (rows == 16) QVGGT_SMALL_ROWS(128, 16); else QVGGT_SMALL_ROWS(128, 32); break;
        case 256: if (rows == 8) QVGGT_SMALL_ROWS(256, 8); else if (rows == 16) QVGGT_SMALL_ROWS(256, 16); else QVGGT_SMALL_ROWS(256, 32); break;
        case 512: if (rows == 8) QVGGT_SMALL_ROWS(512, 8); else QVGGT_SMALL_ROWS(512, 16); break;
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_SMALL_ROWS
#undef QVGGT_SMALL
    return hipGetLastError();
}

}  // namespace qvggt
