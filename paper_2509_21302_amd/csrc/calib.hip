// Calibration side: the reconstruction loss of one quantized linear layer over a calibration batch and its derivatives with
// respect to the smoothing factor and the quantization steps (paper, appendix "Experiment Settings": c_hat and Delta are
// learnable during calibration, learning rates 5e-3 and 5e-2; Sec. 3.1.2, Eq. "loss_ori_overall": squared distance between the
// full-precision and the quantized function over the calibration set).  The paper gives no update rule; the reading is:
//
//   z = (X H) / c,  x_hat = step_x * clamp(round(z / step_x)),      v = (W H) * c,  w_hat[o] = step_w[o] * clamp(round(v[o] / step_w[o])),
//   y_q = x_hat . w_hat^T + b,      L = (1 / T) sum_t || y_q[t] - y_ref[t] ||^2,
//   rounding passed straight through, a clamped value (one whose ROUNDED code leaves the range) passing nothing,
//   d(quantized) / d(step) = round(u) - u inside the range and the clamp bound outside, c_hat moving through both operands (d v / d c = V, d z / d c = -z / c), a dynamic per-token
//   activation step (max |z| / qmax) recomputed from the row and held constant in the derivative, a static one (one value) learnable.
//
// Offline work on batches of a few thousand tokens: codes of both operands once, three matrix products on the bf16 matrix
// instruction (a code is a bf16 number, an fp32 factor is the exact sum of three), the derivatives summed where the products are
// still in registers, and fixed-order sums, so that results do not vary from run to run.
#include "qvggt_common.h"
#include "rotate_rows.h"

#include <algorithm>
#include <type_traits>

namespace qvggt {

namespace {

// ---- X -> X H (orthonormal Hadamard, input-side signs), fp32, natural order: what the loss takes as R and V
template <int K, bool F32>
__global__ __launch_bounds__(256) void rotate_only_kernel(const void *__restrict__ X, int rows, const int8_t *__restrict__ signs,
                                                          float *__restrict__ out)
{
    constexpr int V = RowMap<K>::V, C = RowMap<K>::C, R = RowMap<K>::R;
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), nwaves = gridDim.x * (blockDim.x >> 6);
    const float rs = 1.0f / sqrtf((float)K);
    for (int row = wave; row < rows; row += nwaves) {
        float x[R];
        load_row<K, F32>(X, (size_t)row, lane, x);
        if (signs != nullptr) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int i = 0; i < V; ++i)
                    if (signs[c * 64 * V + lane * V + i] < 0) x[c * V + i] = -x[c * V + i];
        }
        fwht_row<K>(x, lane);
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int i = 0; i < V; ++i) out[(size_t)row * K + c * 64 * V + lane * V + i] = x[c * V + i] * rs;
    }
}

// block-wide sum of one float per thread (256 threads), result in every thread; fixed order
__device__ inline float block_sum(float v, float *red)
{
    v = sum_over_64_lanes(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const float s = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return s;
}

struct QRange {
    float lo, hi;
};

// a product that is not fused with what is added to it
__device__ inline float rounded_product(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}

// the scaled value (a = A / c or A * c): shared by the quantizer and the derivatives, so that both see the same code
__device__ inline float operand_value(float a, float c, bool divide) { return divide ? a / c : a * c; }

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int CT = 128;                  // rows and columns of an output tile; the operands are padded to it with zeros
constexpr float kNothing = __builtin_nanf("");
constexpr int KS1 = 64, KS2 = 32;        // contraction steps of the two GEMM kernels

// ---- codes and steps of both operands.  A fake-quantized value is step * code with a code of at most 8 bits, which bf16 holds
// exactly: the code goes to memory as bf16 (half the bytes of the fp32 product) and the step is applied to the sums.  One wave per
// row: rows 0 .. Tp - 1 are tokens (operand R / c), then Np channels (V * c); rows and columns past the end get zeros, step 0.
// steps[r] is the step the row was quantized with, 0 if there is none (below kMinStep): such a row has codes 0.
// What the products are multiplied by, which takes the quotients that are at hand here, goes to memory with them: by_c[t, j] = -z / c inside the
// range (tokens), by_step[r, j] = d(quantized) / d(step) (channels, and tokens of a static step), and no number where nothing is passed: by_c
// outside the range, both in the padding and in rows without a step.  A derivative by the step is at most 1/2 inside the range and a bound of
// at least 7 outside: it is the mask of a channel's values as well.
__global__ __launch_bounds__(256) void calib_codes_kernel(const float *__restrict__ R, const float *__restrict__ V, const float *__restrict__ c,
                                                          const float *__restrict__ x_step, const float *__restrict__ w_step, QRange q,
                                                          int T, int Tp, int N, int Np, int K, int Kp, uint16_t *__restrict__ codes,
                                                          float *__restrict__ steps, float *__restrict__ by_c, float *__restrict__ by_step_x,
                                                          float *__restrict__ by_step_w)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= Tp + Np) return;
    const bool divide = row < Tp;
    const int r = divide ? row : row - Tp;
    const bool exists = r < (divide ? T : N);
    const float *a = (divide ? R : V) + (size_t)r * K;
    uint16_t *out = codes + (size_t)row * Kp;
    float step = 0.0f;
    if (exists) {
        if (divide && x_step == nullptr) {
            float m = 0.0f;
#pragma unroll 4
            for (int j = 4 * lane; j < K; j += 256) {
                const float4 v = *reinterpret_cast<const float4 *>(a + j);
                m = fmaxf(fmaxf(m, fabsf(operand_value(v.x, c[j], true))), fabsf(operand_value(v.y, c[j + 1], true)));
                m = fmaxf(fmaxf(m, fabsf(operand_value(v.z, c[j + 2], true))), fabsf(operand_value(v.w, c[j + 3], true)));
            }
            m = max_over_64_lanes(m);
            step = m >= q.hi * kMinStep ? m / q.hi : 0.0f;
        } else {
            step = divide ? x_step[0] : w_step[r];
        }
    }
    const bool live = step >= kMinStep;
    if (lane == 0) steps[row] = live ? step : 0.0f;
    float *const bc = divide ? by_c + (size_t)r * Kp : nullptr;
    float *const bs = divide ? (x_step != nullptr ? by_step_x + (size_t)r * Kp : nullptr) : by_step_w + (size_t)r * Kp;
#pragma unroll 4
    for (int j = 4 * lane; j < Kp; j += 256) {
        float code[4] = {0.0f, 0.0f, 0.0f, 0.0f}, dc[4] = {kNothing, kNothing, kNothing, kNothing}, ds[4] = {kNothing, kNothing, kNothing, kNothing};
        if (live && j < K) {
            const float4 v = *reinterpret_cast<const float4 *>(a + j);
            const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = operand_value(x[i], c[j + i], divide), u = z / step, rounded = rintf(u);
                const bool inside = rounded >= q.lo && rounded <= q.hi;
                code[i] = fminf(fmaxf(rounded, q.lo), q.hi);
                ds[i] = inside ? rounded - u : code[i];
                if (divide && inside) dc[i] = -z / c[j + i];
            }
        }
        *reinterpret_cast<uint2 *>(out + j) = make_uint2(pack_bf16x2(code[0], code[1]), pack_bf16x2(code[2], code[3]));
        if (bc != nullptr) *reinterpret_cast<float4 *>(bc + j) = make_float4(dc[0], dc[1], dc[2], dc[3]);
        if (bs != nullptr) *reinterpret_cast<float4 *>(bs + j) = make_float4(ds[0], ds[1], ds[2], ds[3]);
    }
}

// contiguous ranges of work items per XCD (blocks go round-robin over the 8 XCDs): neighbours share operand panels in one L2
__device__ inline int xcd_item(int items)
{
    const int per = (items + 7) >> 3;
    return (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);      // >= items: nothing to do
}

// LDS image of an operand panel of 128 rows: rows of 2 KS bytes, the 16-byte chunks of a row rotated by an XOR so that the 16 rows of
// a fragment read fall into 16 different bank groups
template <int KS>
__device__ inline int panel_offset(int row, int chunk)
{
    return KS == 64 ? row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4) : row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4);
}

// One staged step: acc[mi][ni] += sum over the P pieces of A and the KS contraction indices; a wave owns 64 x 64 of the 128 x 128 tile
template <int KS, int P>
__device__ inline void tile_step(const uint8_t *As, const uint8_t *Bs, int wm, int wn, int lane, v16f (&acc)[2][2])
{
    const int row = lane & 31, half = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < KS / 16; ++ks) {
        v8bf b[2];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) b[ni] = *reinterpret_cast<const v8bf *>(Bs + panel_offset<KS>(wn * 64 + ni * 32 + row, ks * 2 + half));
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const v8bf a = *reinterpret_cast<const v8bf *>(As + p * CT * KS * 2 + panel_offset<KS>(wm * 64 + mi * 32 + row, ks * 2 + half));
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[ni], acc[mi][ni], 0, 0, 0);
            }
    }
}

// row of the tile that register r of sub-tile mi holds (32x32 result layout); the column is wn * 64 + ni * 32 + lane % 32
__device__ inline int tile_row(int wm, int mi, int r, int lane) { return wm * 64 + mi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---- E[t, o] = step_x[t] step_w[o] sum_j qx[t, j] qw[o, j] + b[o] - y_ref[t, o], zero in the padding, and the tile's sum of squares.
// Products of codes are exact, so the only roundings are those of the fp32 accumulation and the epilogue.  Bound by the latency of one
// tile's chain at the sizes of a calibration batch (264 tiles of 16 steps for 1374 x 1024 -> 3072): 26 us there, 298 us as fp32 vector
// tiles.
__global__ __launch_bounds__(256, 2) void calib_residual_kernel(const uint16_t *__restrict__ qx, const uint16_t *__restrict__ qw,
                                                                const float *__restrict__ xs, const float *__restrict__ ws,
                                                                const uint16_t *__restrict__ bias, const float *__restrict__ ref, int T, int N,
                                                                int Kp, int tiles_m, int tiles_n, float *__restrict__ E,
                                                                float *__restrict__ partial)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][2][CT * KS1 * 2];
    __shared__ float red[4];
    const int item = xcd_item(tiles_m * tiles_n);
    if (item >= tiles_m * tiles_n) return;
    const int tm = item % tiles_m, tn = item / tiles_m;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    // eight neighbouring lanes take the 128 bytes of a row (one cache line per row and instruction), 32 rows per pass of the block
    const int lrow = tid >> 3, lch = tid & 7;
    const uint16_t *pa = qx + (size_t)(tm * CT + lrow) * Kp + lch * 8, *pb = qw + (size_t)(tn * CT + lrow) * Kp + lch * 8;
    v4u ra[4], rb[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ra[i] = *reinterpret_cast<const v4u *>(pa + (size_t)(32 * i) * Kp + k0);
            rb[i] = *reinterpret_cast<const v4u *>(pb + (size_t)(32 * i) * Kp + k0);
        }
    };
    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    fetch(0);
    for (int k0 = 0, buf = 0; k0 < Kp; k0 += KS1, buf ^= 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *reinterpret_cast<v4u *>(lds[buf][0] + panel_offset<KS1>(lrow + 32 * i, lch)) = ra[i];
            *reinterpret_cast<v4u *>(lds[buf][1] + panel_offset<KS1>(lrow + 32 * i, lch)) = rb[i];
        }
        fetch(min(k0 + KS1, Kp - KS1));          // the last step's is not used
        __syncthreads();
        tile_step<KS1, 1>(lds[buf][0], lds[buf][1], wm, wn, lane, acc);
    }
    const int Np = tiles_n * CT;
    float sq = 0.0f;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        // all loads of a sub-tile row before the arithmetic, so that they are in flight together
        float rv[2][16], st[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int t = tm * CT + tile_row(wm, mi, r, lane);
            st[r] = xs[t];
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
                rv[ni][r] = ref[(size_t)min(t, T - 1) * N + min(tn * CT + wn * 64 + ni * 32 + (lane & 31), N - 1)];
        }
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            const int o = tn * CT + wn * 64 + ni * 32 + (lane & 31);
            const float so = ws[o], bo = bias != nullptr ? bf16_bits_to_float(bias[min(o, N - 1)]) : 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = tm * CT + tile_row(wm, mi, r, lane);
                float v = acc[mi][ni][r] * st[r] * so;
                if (bias != nullptr) v += bo;
                v -= rv[ni][r];
                v = (t < T && o < N) ? v : 0.0f;
                sq = fmaf(v, v, sq);
                E[(size_t)t * Np + o] = v;
            }
        }
    }
    sq = block_sum(sq, red);
    if (tid == 0) partial[item] = sq;
}

// ---- the two products with E and what is summed over them.
//   GX[t, j] = sum_o (E[t, o] step_w[o]) qw[o, j],     GW[o, j] = sum_t (E[t, o] step_x[t]) qx[t, j]
// Neither is stored: the derivatives are linear in them, so a block multiplies its piece of GX or GW (one tile, one share of the
// contraction) by the masks and step derivatives that calib_codes_kernel left, and leaves sums over its rows and columns:
//   dL / d c[j]       <-  sum_o GW [inside] V  +  sum_t GX [inside] (-z / c)
//   dL / d step_w[o]  <-  sum_j GW d(hat) / d(step)          dL / d step_x  <-  sum_t,j GX d(hat) / d(step)   (static step)
// The fp32 factor E * step is split into three bf16 numbers of 8 significant bits each, which add up to it exactly, and a code is a
// bf16 number: three bf16 MFMAs give the products of the fp32 value and the code without rounding, at five times the rate of the
// fp32 matrix instruction.  Measured at 1374 x 1024 -> 3072: 84 us, 0.63 PFLOP/s of bf16 MFMAs.  No unit is full (MFMA 26 %, vector ALU 39 %, LDS 24 % of
// the cycles): the parts of a step, loads, splitting, LDS and MFMAs, share two waves per SIMD (switched off one by one in a copy: 64 us without
// the loads, 73 without the splitting, 62 without the MFMAs; 67 without the sums at the end of a tile).  With the masks and quotients computed
// in those sums it was 113 us, as fp32 vector tiles that stored GX and GW 815 and the derivatives' own passes over them 901.
struct CalibPlan {
    int Tp, Np, Kp, tm, tn, tj;         // padded sizes and their 128-tiles
    int chunk_x, split_x;               // contraction of GX (over channels): length of a share, shares
    int chunk_w, split_w;               // contraction of GW (over tokens)
    int items_x, items_w;
};

__global__ __launch_bounds__(256, 2) void calib_products_kernel(const float *__restrict__ E, const uint16_t *__restrict__ qx,
                                                                const uint16_t *__restrict__ qw, const float *__restrict__ xs,
                                                                const float *__restrict__ ws, const float *__restrict__ V,
                                                                const float *__restrict__ by_c, const float *__restrict__ by_step_x,
                                                                const float *__restrict__ by_step_w, int N, int K, CalibPlan pl,
                                                                bool want_step_x, float *__restrict__ part_c,
                                                                float *__restrict__ part_w, float *__restrict__ part_x)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][4][CT * KS2 * 2];       // three pieces of A, then B
    __shared__ float colsum[2][CT], rowsum[2][CT], red[4];
    int item = xcd_item(pl.items_x + pl.items_w);
    if (item >= pl.items_x + pl.items_w) return;
    const bool is_x = item < pl.items_x;
    const int first = is_x ? 0 : pl.items_x;
    item -= first;
    const int tj = item % pl.tj, rest = item / pl.tj;
    const int split = is_x ? pl.split_x : pl.split_w;
    const int tm = rest / split, sp = rest % split;
    const int len = is_x ? pl.Np : pl.Tp, chunk = is_x ? pl.chunk_x : pl.chunk_w;
    const int kb = sp * chunk, ke = min(kb + chunk, len);
    const uint16_t *qb = (is_x ? qw : qx) + tj * CT;
    const float *ks = is_x ? ws : xs;                       // step that goes with the contraction index
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;

    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // The two products differ in which index of E is the contraction.  Each has its own loop: what is fetched for the steps ahead stays as loaded
    // until it is staged, a step later, so that nothing in between waits for memory.  (With the two kinds of fetch as branches of one loop, and the
    // steps applied in them, every step waited for its loads: 90 us of products at 1374 x 1024 -> 3072, 81 this way.  Two steps ahead: no faster.)
    auto contract = [&](auto is_x_c) {
        constexpr bool IS_X = decltype(is_x_c)::value;
        float fa[16], st[IS_X ? 4 : 8];                     // E as loaded, the steps that go with it
        uint32_t rb[8];                                     // B: codes of columns 2 lane, 2 lane + 1 at eight contraction indices
        // one running pointer per operand: tokens as rows take four channels of rows tid / 8 + 32 i (a line per row), channels as rows
        // 2 lane, 2 lane + 1 eight consecutive tokens of each
        const float *e0 = IS_X ? E + (size_t)(tm * CT + (tid >> 3)) * pl.Np + (tid & 7) * 4 : E + (size_t)(wave * 8) * pl.Np + tm * CT + 2 * lane;
        const uint16_t *b0 = qb + (size_t)(wave * 8) * pl.Kp + 2 * lane;
        auto fetch = [&](int k0) {
            if constexpr (IS_X) {
                const float4 w = *reinterpret_cast<const float4 *>(ks + k0 + (tid & 7) * 4);
                st[0] = w.x; st[1] = w.y; st[2] = w.z; st[3] = w.w;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 v = *reinterpret_cast<const float4 *>(e0 + (size_t)(32 * i) * pl.Np + k0);
                    fa[4 * i] = v.x; fa[4 * i + 1] = v.y; fa[4 * i + 2] = v.z; fa[4 * i + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float2 v = *reinterpret_cast<const float2 *>(e0 + (size_t)(k0 + i) * pl.Np);
                    st[i] = ks[k0 + wave * 8 + i];
                    fa[i] = v.x; fa[8 + i] = v.y;
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) rb[i] = *reinterpret_cast<const uint32_t *>(b0 + (size_t)(k0 + i) * pl.Kp);
        };
        auto stage = [&](int buf) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {                   // eight values: four of rows 2 h, 2 h + 1 of this thread, or a chunk of row 2 lane + h
                uint32_t w[3][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t hi[2], mid[2], low[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int n = 2 * i + e;
                        const float f = rounded_product(fa[8 * h + n], st[IS_X ? n % 4 : n]);
                        hi[e] = __float_as_uint(f);
                        float rem = f - __uint_as_float(hi[e] & 0xFFFF0000u);
                        rem = rem == rem ? rem : 0.0f;      // an infinite f is its own first piece
                        mid[e] = __float_as_uint(rem);
                        low[e] = __float_as_uint(rem - __uint_as_float(mid[e] & 0xFFFF0000u));
                    }
                    w[0][i] = __builtin_amdgcn_perm(hi[1], hi[0], 0x07060302);
                    w[1][i] = __builtin_amdgcn_perm(mid[1], mid[0], 0x07060302);
                    w[2][i] = __builtin_amdgcn_perm(low[1], low[0], 0x07060302);
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    if constexpr (IS_X) {
                        const int row = (tid >> 3) + 64 * h, ch = (tid & 7) >> 1, half = (tid & 1) * 8;
                        *reinterpret_cast<uint2 *>(lds[buf][p] + panel_offset<KS2>(row, ch) + half) = make_uint2(w[p][0], w[p][1]);
                        *reinterpret_cast<uint2 *>(lds[buf][p] + panel_offset<KS2>(row + 32, ch) + half) = make_uint2(w[p][2], w[p][3]);
                    } else {
                        *reinterpret_cast<uint4 *>(lds[buf][p] + panel_offset<KS2>(2 * lane + h, wave)) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
                    }
                }
                uint32_t b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) b[i] = __builtin_amdgcn_perm(rb[2 * i + 1], rb[2 * i], h == 0 ? 0x05040100 : 0x07060302);
                *reinterpret_cast<uint4 *>(lds[buf][3] + panel_offset<KS2>(2 * lane + h, wave)) = make_uint4(b[0], b[1], b[2], b[3]);
            }
        };
        fetch(kb);
        for (int k0 = kb, buf = 0; k0 < ke; k0 += KS2, buf ^= 1) {
            stage(buf);
            fetch(min(k0 + KS2, ke - KS2));          // the last step's is not used
            __syncthreads();
            tile_step<KS2, 3>(lds[buf][0], lds[buf][3], wm, wn, lane, acc);
        }
    };
    if (is_x) contract(std::true_type{});
    else contract(std::false_type{});

    // sums over the tile's columns (dL / dc) and rows (dL / d step)
    float col[2] = {0.0f, 0.0f}, rowv[2][16], all = 0.0f;
    const int j0 = tj * CT + wn * 64 + (lane & 31);
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        // what the products are multiplied by: loads first, in flight together
        float dc[2][16], ds[2][16];
        if (is_x) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const size_t at = (size_t)(tm * CT + tile_row(wm, mi, r, lane)) * pl.Kp + j0;
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    dc[ni][r] = by_c[at + 32 * ni];
                    ds[ni][r] = want_step_x ? by_step_x[at + 32 * ni] : kNothing;
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = tm * CT + tile_row(wm, mi, r, lane);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    dc[ni][r] = V[(size_t)min(m, N - 1) * K + min(j0 + 32 * ni, K - 1)];
                    ds[ni][r] = by_step_w[(size_t)m * pl.Kp + j0 + 32 * ni];
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) dc[ni][r] = fabsf(ds[ni][r]) <= 0.5f ? dc[ni][r] : kNothing;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float s = 0.0f;
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
                const float g = acc[mi][ni][r];
                col[ni] = dc[ni][r] == dc[ni][r] ? fmaf(g, dc[ni][r], col[ni]) : col[ni];
                s = ds[ni][r] == ds[ni][r] ? fmaf(g, ds[ni][r], s) : s;
            }
            rowv[mi][r] = s;
        }
    }
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
        col[ni] += __shfl_xor(col[ni], 32);
        if (lane < 32) colsum[wm][wn * 64 + ni * 32 + lane] = col[ni];
    }
    if (!is_x) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float v = rowv[mi][r];
                v = dpp_add_step<0xB1>(v); v = dpp_add_step<0x4E>(v); v = dpp_add_step<0x141>(v); v = dpp_add_step<0x140>(v);
                v += __shfl_xor(v, 16);
                if ((lane & 31) == 0) rowsum[wn][tile_row(wm, mi, r, lane)] = v;
            }
    } else if (want_step_x) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) all += rowv[mi][r];
    }
    __syncthreads();
    const int part = (is_x ? 0 : pl.tm * pl.split_x) + rest;
    if (tid < CT) {
        part_c[(size_t)part * pl.Kp + tj * CT + tid] = colsum[0][tid] + colsum[1][tid];
        if (!is_x) part_w[(size_t)(tj * split + sp) * pl.Np + tm * CT + tid] = rowsum[0][tid] + rowsum[1][tid];
    }
    if (is_x && want_step_x) {
        all = block_sum(all, red);
        if (tid == 0) part_x[item] = all;
    }
}

// ---- the partial sums of all blocks, added in a fixed order and in double: 16 columns of grad_c per block, then 16 channels of
// grad_w per block (16 groups of threads share the parts), then one block each for the loss and the derivative of a static step
__global__ __launch_bounds__(256) void calib_sums_kernel(const float *__restrict__ part_c, const float *__restrict__ part_w,
                                                         const float *__restrict__ part_x, const float *__restrict__ part_loss, int N, int K,
                                                         CalibPlan pl, float scale, float loss_scale, float *__restrict__ grad_c,
                                                         float *__restrict__ grad_w, float *__restrict__ grad_x, float *__restrict__ loss)
{
    __shared__ double red[256];
    const int tid = threadIdx.x, blocks_c = (K + 15) / 16, blocks_w = (N + 15) / 16;
    const int b = blockIdx.x;
    const bool vec = b < blocks_c + blocks_w, is_c = b < blocks_c, is_loss = b == blocks_c + blocks_w;
    const int col = vec ? (is_c ? b : b - blocks_c) * 16 + (tid & 15) : 0;
    const float *part = vec ? (is_c ? part_c : part_w) + col : is_loss ? part_loss : part_x;
    const size_t pitch = vec ? (is_c ? pl.Kp : pl.Np) : 1;
    const int n = vec ? (is_c ? pl.tm * pl.split_x + pl.tn * pl.split_w : pl.tj * pl.split_w) : (is_loss ? pl.tm * pl.tn : pl.items_x);
    double s = 0.0;
#pragma unroll 8
    for (int p = vec ? tid >> 4 : tid; p < n; p += vec ? 16 : 256) s += (double)part[p * pitch];
    red[tid] = s;
    __syncthreads();
    for (int h = 128; h >= (vec ? 16 : 1); h >>= 1) {
        if (tid < h) red[tid] += red[tid + h];
        __syncthreads();
    }
    if (vec) {
        if (tid < 16 && col < (is_c ? K : N)) (is_c ? grad_c : grad_w)[col] = (float)(red[tid] * (double)scale);
    } else if (tid == 0) {
        (is_loss ? loss : grad_x)[0] = (float)(red[0] * (double)(is_loss ? loss_scale : scale));
    }
}

__global__ void descent_step_kernel(float *__restrict__ theta, const float *__restrict__ grad, int n, float lr, float floor_)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) theta[i] = fmaxf(theta[i] - lr * grad[i], floor_);
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

hipError_t run_rotate_only(const void *X, bool f32, int rows, int K, const int8_t *signs, float *out, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    const int blocks = std::min((rows + 3) / 4, 2048);
#define QVGGT_ROT(KK)                                                                                          \
    case KK:                                                                                                   \
        if (f32) rotate_only_kernel<KK, true><<<blocks, 256, 0, stream>>>(X, rows, signs, out);               \
        else rotate_only_kernel<KK, false><<<blocks, 256, 0, stream>>>(X, rows, signs, out);                  \
        break;
    switch (K) {
        QVGGT_ROT(128) QVGGT_ROT(256) QVGGT_ROT(512) QVGGT_ROT(1024) QVGGT_ROT(2048) QVGGT_ROT(4096) QVGGT_ROT(8192)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_ROT
    return hipGetLastError();
}

// Shares of the two contractions.  A block's work is one 128 x 128 tile over one share; 512 blocks are resident (two per compute unit),
// and since the results are linear in the products a contraction may be cut anywhere.  Of the share lengths that are multiples of
// 128 the one with the least (rounds of 512 blocks) x (length + 96) is used: a tile's epilogue takes about as long as 96 contraction
// indices, three of the kernel's steps.
static CalibPlan calib_plan(int T, int N, int K)
{
    CalibPlan p;
    auto up = [](int v) { return (v + CT - 1) / CT * CT; };
    p.Tp = up(T); p.Np = up(N); p.Kp = up(K);
    p.tm = p.Tp / CT; p.tn = p.Np / CT; p.tj = p.Kp / CT;
    long long best = -1;
    int best_len = CT;
    const int longest = std::max(p.Tp, p.Np);
    for (int len = CT; len <= longest && len <= 64 * CT; len += CT) {
        const long long blocks = (long long)p.tm * p.tj * ((p.Np + len - 1) / len) + (long long)p.tn * p.tj * ((p.Tp + len - 1) / len);
        const long long cost = (blocks + 511) / 512 * (len + 96);
        if (best < 0 || cost < best) { best = cost; best_len = len; }
    }
    auto shares = [&](int total, int &chunk, int &split) {
        split = (total + best_len - 1) / best_len;
        chunk = ((total + split - 1) / split + KS2 - 1) / KS2 * KS2;
        split = (total + chunk - 1) / chunk;
    };
    shares(p.Np, p.chunk_x, p.split_x);
    shares(p.Tp, p.chunk_w, p.split_w);
    p.items_x = p.tm * p.tj * p.split_x;
    p.items_w = p.tn * p.tj * p.split_w;
    return p;
}

// workspace: codes of both operands [Tp + Np, Kp] bf16, their steps [Tp + Np], what the products are multiplied by (up to [2 Tp + Np, Kp]), E
// [Tp, Np], partial sums: 52 of the 53 MB that are asked for at 1374 x 1024 -> 3072.  Tp x Kp of them are a static step's alone; with z in place of both
// of its planes and the quotients taken again in the products, 2748 x 4096 -> 64 asks for 93 MB and not 121, and takes 141 us and not 129
// (1374 x 1024 -> 3072 138 and not 120).  The size has always covered fp32 copies of both operands,
// both products and E, the ABI's tests hold it to that, and it stays where the own need is less.
size_t calib_workspace_bytes(int T, int N, int K)
{
    const CalibPlan p = calib_plan(T, N, K);
    const size_t own = align256((size_t)(p.Tp + p.Np) * p.Kp * 2) + 2 * align256((size_t)p.Tp * p.Kp * 4) + align256((size_t)p.Np * p.Kp * 4) + align256((size_t)(p.Tp + p.Np) * 4) + align256((size_t)p.Tp * p.Np * 4) +
                       align256(((size_t)p.tm * p.split_x + (size_t)p.tn * p.split_w) * p.Kp * 4) + align256((size_t)p.tj * p.split_w * p.Np * 4) +
                       align256((size_t)p.items_x * 4) + align256((size_t)p.tm * p.tn * 4);
    return std::max(own, 4 * (2 * (size_t)T * K + 2 * (size_t)N * K + (size_t)T * N));
}

hipError_t run_calib_loss_grad(const float *R, const float *V, const float *y_ref, const void *bias, const float *c_hat,
                               const float *w_step, const float *x_step, int T, int N, int K, int bits, float *loss, float *grad_c,
                               float *grad_w_step, float *grad_x_step, void *workspace, hipStream_t stream)
{
    const CalibPlan pl = calib_plan(T, N, K);
    uint8_t *p = static_cast<uint8_t *>(workspace);
    auto take = [&](size_t bytes) { uint8_t *r = p; p += align256(bytes); return r; };
    uint16_t *codes = reinterpret_cast<uint16_t *>(take((size_t)(pl.Tp + pl.Np) * pl.Kp * 2));
    float *steps = reinterpret_cast<float *>(take((size_t)(pl.Tp + pl.Np) * 4));
    float *by_c = reinterpret_cast<float *>(take((size_t)pl.Tp * pl.Kp * 4)), *by_step_x = reinterpret_cast<float *>(take((size_t)pl.Tp * pl.Kp * 4));
    float *by_step_w = reinterpret_cast<float *>(take((size_t)pl.Np * pl.Kp * 4));
    float *E = reinterpret_cast<float *>(take((size_t)pl.Tp * pl.Np * 4));
    float *part_c = reinterpret_cast<float *>(take(((size_t)pl.tm * pl.split_x + (size_t)pl.tn * pl.split_w) * pl.Kp * 4));
    float *part_w = reinterpret_cast<float *>(take((size_t)pl.tj * pl.split_w * pl.Np * 4));
    float *part_x = reinterpret_cast<float *>(take((size_t)pl.items_x * 4));
    float *part_loss = reinterpret_cast<float *>(take((size_t)pl.tm * pl.tn * 4));
    const uint16_t *qx = codes, *qw = codes + (size_t)pl.Tp * pl.Kp;
    const float *xs = steps, *ws = steps + pl.Tp;
    const QRange q{-(float)(1 << (bits - 1)), (float)((1 << (bits - 1)) - 1)};
    const float scale = 2.0f / (float)T;                 // dL / dy_q = (2 / T) E: folded into the last sums
    auto grid8 = [](int items) { return (unsigned)((items + 7) / 8 * 8); };

    calib_codes_kernel<<<(pl.Tp + pl.Np) / 4, 256, 0, stream>>>(R, V, c_hat, x_step, w_step, q, T, pl.Tp, N, pl.Np, K, pl.Kp, codes, steps, by_c, by_step_x,
                                                                        by_step_w);
    calib_residual_kernel<<<grid8(pl.tm * pl.tn), 256, 0, stream>>>(qx, qw, xs, ws, reinterpret_cast<const uint16_t *>(bias), y_ref, T, N, pl.Kp,
                                                                   pl.tm, pl.tn, E, part_loss);
    const bool static_step = x_step != nullptr;
    calib_products_kernel<<<grid8(pl.items_x + pl.items_w), 256, 0, stream>>>(E, qx, qw, xs, ws, V, by_c, by_step_x, by_step_w, N, K, pl, static_step, part_c,
                                                                             part_w, part_x);
    calib_sums_kernel<<<(K + 15) / 16 + (N + 15) / 16 + 1 + static_step, 256, 0, stream>>>(part_c, part_w, part_x, part_loss, N, K, pl, scale,
                                                                                             1.0f / (float)T, grad_c, grad_w_step, grad_x_step, loss);
    return hipGetLastError();
}

hipError_t run_descent_step(float *theta, const float *grad, int n, float lr, float floor_, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    descent_step_kernel<<<(n + 255) / 256, 256, 0, stream>>>(theta, grad, n, lr, floor_);
    return hipGetLastError();
}

}  // namespace qvggt
