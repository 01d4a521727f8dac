// Kernel 1 on the matrix cores for many bf16 rows of K = 2^n * m values, m = 12 or 20 (a Paley factor), and of K = 8192 (H_16 in its
// place).  Few rows, fp32 ones, weights, the column
// statistic and the other sizes are in rotate_quant_general.hip, resp. rotate_quant.hip.
//
// H_K = H_{K / S} (x) (H_8 (x) H_m), S = 8 m = 96, 160 or 128.  A row is a (K / S) x S matrix of segments; its product with the right factor is taken
// on the matrix cores: the inputs and the +-1 entries are exact bf16 operands, the sums accumulate in fp32, and S is whole in 32-column
// tiles where m itself would leave lanes idle.  The left factor is 3 to 6 butterfly stages between the accumulator registers, as in
// rotate_quant_mfma.hip, whose order of MFMA rows this kernel has.
//
// Order of the contraction: a k-step of 16 is four values of b (4 q ..) for four values of the segment's three-bit index a (bit 2: the step,
// bit 1: the lane half, bit 0: the operand's two pieces of 8 bytes); a column tile is four outputs b' (4 nt ..) for all eight a'.  The operand
// of the +-1 entries then depends on the step only through q, and through the sign of bit 2 of a' (one xor): m^2 / 16 fragments instead of twice as many,
// in registers for m = 12 (36; at K = 6144 there is no room), in LDS otherwise (25 KiB, m = 16: 16).
//
// Codes are in natural order (element e at position e).  A lane's results are one column of all segments; its codes go to LDS one by one, where the row's
// input was, and leave from there in whole units (E2M3: staged as bf16 numbers, which a conversion takes 32 at a time; converting staged bytes
// took 5 vector instructions a code instead of 2) or 16-byte pieces of a row.
//
// Bound by the vector ALU (12 to 14 instructions a value) up to K = 1536 and by it and memory beyond: 16384 rows to E2M3, us of the general kernel / this one,
// K = 768 18.0 / 14.8 (2.3 TB/s), 1536 29.5 / 23.9, 3072 69.0 / 36.1 (3.8 TB/s), 6144 148 / 82, 2560 51.9 / 32.6, 5120 110 / 66.8.  With two waves per SIMD
// throughout: m = 20 and K = 6144 with one wave per SIMD took 41.0, 76.7 and 87.1.
#include "paley.h"
#include "qvggt_common.h"
#include "rotate_rows.h"

#include <algorithm>
#include <climits>
#include <utility>

namespace qvggt {

namespace pal {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

template <int MM, int HB>
struct Cfg {
    static constexpr int S = 8 * MM, K = S * HB, NT = MM / 4;         // segment, row, column tiles
    static constexpr int RT = HB > 32 ? 2 : 1;                        // row tiles of 32 segments that a wave works on
    static constexpr int TOK = 32 * RT / HB;                          // tokens of a wave's tile
    static constexpr int T = HB == 8 ? 2 : 1;                         // tokens a lane sees in its registers
    static constexpr int HBL = HB == 8 ? 8 : 16;                      // segments per lane, token and row tile
    static constexpr int LOADS = RT * S / 16;                         // 16-byte loads per lane and tile
    static constexpr int SIGN_CLASSES = K % 512 == 0 ? K / 512 : K / 256;
    static constexpr int PITCH = 2 * S + 16;                          // of a staged segment: four times an odd number of banks
    static constexpr int WAVE_LDS = 32 * RT * PITCH;
    // What a wave has no registers for beside another on its SIMD is in LDS, and where two blocks do not fit there a block has eight waves
    static constexpr bool SHARED = HB == 64 || (MM == 20 && HB >= 16);
    static constexpr int WAVES = SHARED && MM != 16 ? 8 : 4;          // eight waves' rows of 8192 values are 136 KiB and the tables 48
    static constexpr int BLOCKS_PER_CU = SHARED ? 1 : 2, WAVES_PER_SIMD = WAVES * BLOCKS_PER_CU / 4;
    static constexpr bool TABLES_IN_LDS = MM != 12 || SHARED;         // the +-1 fragments and the multipliers
    static constexpr int FRAGMENTS_AT = WAVES * WAVE_LDS, MULTIPLIERS_AT = FRAGMENTS_AT + (TABLES_IN_LDS ? NT * NT * 1024 : 0);
    static constexpr int LDS_BYTES = MULTIPLIERS_AT + (TABLES_IN_LDS ? K * 4 : 0);
    static_assert(LDS_BYTES * BLOCKS_PER_CU <= 160 * 1024, "the blocks of a compute unit share its LDS");
    static_assert(LOADS % SIGN_CLASSES == 0 && LOADS % NT == 0, "sign masks and staging addresses repeat with whole loads");
};

// bit b' of neg_row<MM>(b): entry (b, b') is -1
template <int MM>
constexpr uint32_t neg_row(int b)
{
    uint32_t m = 0;
    for (int c = 0; c < MM; ++c)
        if constexpr (MM == 16) m |= (uint32_t)(__builtin_popcount(b & c) & 1) << c;      // the power of two: H_16
        else m |= (gen::paley_entry<MM>(b, c) < 0 ? 1u : 0u) << c;
    return m;
}
template <int MM>
struct NegRows {
    uint32_t row[MM];
    constexpr NegRows() : row()
    {
        for (int b = 0; b < MM; ++b) row[b] = neg_row<MM>(b);
    }
};

// MFMA row m of a row tile -> segment of the tile (token * HB + hb, or hb mod 32)
template <int HB>
__device__ inline int segment_of_row(int m)
{
    if (HB == 8) return (m & 3) | (m >> 3 & 1) << 2 | (m >> 2 & 1) << 3 | (m >> 4 & 1) << 4;      // hb0, hb1, hb2, tk0, tk1
    return (m & 3) | (m >> 3 & 3) << 2 | (m >> 2 & 1) << 4;                                       // hb0 .. hb3, hb4 or tk0
}

}  // namespace pal

// CB: 4 packed nibbles, 8 int8 rows, 6 E2M3 blocks.  mul, step and qmax as rotate_rows_general_kernel.
template <int MM, int HB, int CB>
__global__ __launch_bounds__((pal::Cfg<MM, HB>::WAVES * 64), (pal::Cfg<MM, HB>::WAVES_PER_SIMD)) void rotate_quant_paley_kernel(
    const uint16_t *__restrict__ X, int rows, const int8_t *__restrict__ signs, const float *__restrict__ mul,
    uint8_t *__restrict__ out, float *__restrict__ scale, const float *__restrict__ step, int step_stride, float qmax)
{
    using namespace pal;
    using C = Cfg<MM, HB>;
    constexpr int K = C::K, NT = C::NT, RT = C::RT, TOK = C::TOK, WAVES = C::WAVES;
    constexpr bool BLOCK_FLUSH = CB == 6 && TOK == 1;          // the block's rows leave together: runs of 48 bytes per row and unit
    constexpr bool WIDE = CB == 6;                    // codes are staged as bf16 numbers, which a conversion takes 32 at a time; bytes otherwise
    constexpr int CODE_BYTES = WIDE ? 2 : 1, CODE_PITCH = CODE_BYTES * K + 16;        // of a staged row of codes
    static_assert(TOK * CODE_PITCH <= C::WAVE_LDS, "a tile's codes fit its staging rows");
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::LDS_BYTES];
    const int lane = threadIdx.x & 63, wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 31, g = lane >> 5, a_out = c >> 2, j_out = c & 3;
    uint8_t *const lds = smem + wave_in_block * C::WAVE_LDS;
    uint8_t *const fragments = smem + C::FRAGMENTS_AT;
    float4 *const multipliers = reinterpret_cast<float4 *>(smem + C::MULTIPLIERS_AT);
    const int wave = (int)blockIdx.x * WAVES + wave_in_block, nwaves = (int)gridDim.x * WAVES;
    const int ntiles = (rows + TOK - 1) / TOK;

    // ---- loads: a tile is 32 * RT * S consecutive values
    const size_t max_flat = (size_t)rows * K;
    auto load16 = [&](const uint16_t *p) -> uint4 {            // X is read once: past the caches
        const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p));
        return make_uint4(v[0], v[1], v[2], v[3]);
    };
    uint4 G[C::LOADS];
    auto load_tile = [&](int t) {
        if ((t + 1) * TOK <= rows) {
            const uint16_t *p = X + (size_t)t * (TOK * K) + 8 * lane;
#pragma unroll
            for (int j = 0; j < C::LOADS; ++j) G[j] = load16(p + 512 * j);
        } else {                                               // rows past the end: the last row again, not written
#pragma unroll
            for (int j = 0; j < C::LOADS; ++j) {
                size_t f = (size_t)t * (TOK * K) + 512 * j + 8 * lane;
                if (f >= max_flat) f = max_flat - K + f % K;
                G[j] = load16(X + f);
            }
        }
    };
    int tile = wave;
    if (tile < ntiles) {
        load_tile(tile);
    } else if constexpr (BLOCK_FLUSH) {
#pragma unroll
        for (int j = 0; j < C::LOADS; ++j) G[j] = make_uint4(0u, 0u, 0u, 0u);
    }

    // ---- per-lane constants: all loads first, then what needs none of them, then the arithmetic on them
    uint2 sb[C::SIGN_CLASSES];
#pragma unroll
    for (int q = 0; q < C::SIGN_CLASSES; ++q) sb[q] = signs != nullptr ? *reinterpret_cast<const uint2 *>(signs + (512 * q + 8 * lane) % K) : make_uint2(0u, 0u);
    // multipliers of the lane's results: register r of row tile rt, column tile nt; in LDS four registers of a lane together
    auto element = [&](int rt, int r, int nt, int l) {
        const int hb = HB >= 32 ? (r & 7) | ((l >> 5) << 3) | ((r >> 3) << 4) | (rt << 5) : r;
        return (hb * 8 + ((l & 31) >> 2)) * MM + 4 * nt + (l & 3);
    };
    constexpr bool IN_LDS = C::TABLES_IN_LDS;
    constexpr int CM_LANES = HB >= 32 ? 64 : 32, CM_FOURS = C::HBL / 4;
    constexpr int CMS = IN_LDS ? K / (WAVES * 64) : RT * C::HBL * NT;         // multipliers that a lane loads
    static_assert(RT * NT * C::HBL * CM_LANES == K && CMS * (IN_LDS ? WAVES * 64 : CM_LANES) == K, "every multiplier once");
    float cm[CMS];
    const float rs = 1.0f / sqrtf((float)K);
#pragma unroll
    for (int i = 0; i < CMS; ++i) {
        int e;
        if constexpr (IN_LDS) {
            const int at = i * WAVES * 64 + (int)threadIdx.x, l = (at >> 2) % CM_LANES, k = (at >> 2) / CM_LANES;
            e = element(k / CM_FOURS / NT, 4 * (k % CM_FOURS) + (at & 3), k / CM_FOURS % NT, l);
        } else {
            e = element(i / (C::HBL * NT), i / NT % C::HBL, i % NT, lane);
        }
        cm[i] = mul != nullptr ? mul[e] : rs;
    }
    // fragments of the +-1 entries for bit 2 of a = 0: element i (piece p = i / 4, value 4 q + i % 4) of the lane's column
    constexpr NegRows<MM> neg;
    v4u frag[IN_LDS ? 1 : NT * NT];
    {
        const uint32_t one[2] = {0x3F803F80u ^ ((__popc((2 * g) & a_out) & 1) ? 0x80008000u : 0u), 0x3F803F80u ^ ((__popc((2 * g + 1) & a_out) & 1) ? 0x80008000u : 0u)};
        auto fragment = [&](int q, int nt) {
            v4u w;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int b = 4 * q + 2 * (d & 1);
                w[d] = one[d >> 1] ^ ((neg.row[b] >> (4 * nt + j_out) & 1u) << 15) ^ ((neg.row[b + 1] >> (4 * nt + j_out)) << 31);
            }
            return w;
        };
        if constexpr (IN_LDS) {
#pragma unroll
            for (int f = 0; f < NT * NT; ++f)
                if (f % WAVES == wave_in_block) *reinterpret_cast<v4u *>(fragments + f * 1024 + lane * 16) = fragment(f / NT, f % NT);
        } else {
#pragma unroll
            for (int f = 0; f < NT * NT; ++f) frag[f] = fragment(f / NT, f % NT);
        }
    }
    uint32_t sgn[C::SIGN_CLASSES][4];                          // load j: sign masks of class j % SIGN_CLASSES
#pragma unroll
    for (int q = 0; q < C::SIGN_CLASSES; ++q) {
        const uint32_t w[2] = {sb[q].x, sb[q].y};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t two = w[d >> 1] >> (16 * (d & 1));
            sgn[q][d] = ((two & 0x80u) << 8) | ((two & 0x8000u) << 16);
        }
    }
    if constexpr (IN_LDS) {
#pragma unroll
        for (int i = 0; i < CMS; ++i) reinterpret_cast<float *>(multipliers)[i * WAVES * 64 + threadIdx.x] = cm[i];
        __syncthreads();
    }
    const uint32_t flip = (c & 16) ? 0x80008000u : 0u;         // bit 2 of a = 1: columns with bit 2 of a' the other way
    // staging: 16-byte piece 64 j + lane of the tile; NT loads are 16 segments
    uint32_t wr[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int id = 64 * j + lane;
        wr[j] = id / (C::S / 8) * C::PITCH + id % (C::S / 8) * 16;
    }
    const int rd = segment_of_row<HB>(c) * C::PITCH + g * 4 * MM;
    // codes: position 4 nt + j of segment hb(r), a_out
    const int code_lane = CODE_BYTES * (a_out * MM + j_out) + g * (HB >= 32 ? CODE_BYTES * 64 * MM : CODE_PITCH);
    const int q_hi = (int)qmax, q_lo = -q_hi - 1;

    for (; (BLOCK_FLUSH ? tile - wave_in_block : tile) < ntiles; tile += nwaves) {
#pragma unroll
        for (int j = 0; j < C::LOADS; ++j) {
            const int q = j % C::SIGN_CLASSES;
            uint4 v = G[j];
            v.x ^= sgn[q][0]; v.y ^= sgn[q][1]; v.z ^= sgn[q][2]; v.w ^= sgn[q][3];
            *reinterpret_cast<uint4 *>(lds + wr[j % NT] + j / NT * 16 * C::PITCH) = v;
        }
        lanes_exchange_fence();
        if (tile + nwaves < ntiles) load_tile(tile + nwaves);

        v16f acc[RT][NT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[rt][nt][r] = 0.0f;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            v4u b[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                b[nt] = IN_LDS ? *reinterpret_cast<const v4u *>(fragments + (q * NT + nt) * 1024 + lane * 16) : frag[IN_LDS ? 0 : q * NT + nt];
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint8_t *p = lds + rd + rt * 32 * C::PITCH + hi * 8 * MM + 8 * q;
                    const v2u p0 = *reinterpret_cast<const v2u *>(p), p1 = *reinterpret_cast<const v2u *>(p + 2 * MM);
                    const v4u a = {p0[0], p0[1], p1[0], p1[1]};
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if (hi == 1 && rt == 0) b[nt] = b[nt] ^ flip;
                        acc[rt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b[nt]), acc[rt][nt], 0, 0, 0);
                    }
                }
            }
        }
        // H_{K / S} over the segments: register bits 0, 1, 2, (3), the lane half, the row tile
        constexpr int REG_STAGES = HB >= 16 ? 4 : 3;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                for (int s = 0; s < REG_STAGES; ++s) {
                    const int h = 1 << s;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if ((r & h) == 0) {
                            const float a = acc[rt][nt][r], d = acc[rt][nt][r + h];
                            acc[rt][nt][r] = a + d;
                            acc[rt][nt][r + h] = a - d;
                        }
                }
                if constexpr (HB >= 32) {
                    // hb bit 4 is the lane half: halves are swapped between registers r and r + 8 (register bit 3 means hb4 then, the lane half hb3)
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[rt][nt][r]), __float_as_uint(acc[rt][nt][r + 8]), false, false);
                        const float a = __uint_as_float(sw[0]), d = __uint_as_float(sw[1]);
                        acc[rt][nt][r] = a + d;
                        acc[rt][nt][r + 8] = a - d;
                    }
                }
            }
            if constexpr (RT == 2) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float a = acc[0][nt][r], d = acc[RT - 1][nt][r];
                    acc[0][nt][r] = a + d;
                    acc[RT - 1][nt][r] = a - d;
                }
            }
        }
        float amax[C::T];
#pragma unroll
        for (int t = 0; t < C::T; ++t) amax[t] = 0.0f;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float m[4];
                    if constexpr (IN_LDS) {
                        const float4 v = multipliers[((rt * NT + nt) * CM_FOURS + k % CM_FOURS) * CM_LANES + (HB >= 32 ? lane : c)];
                        m[0] = v.x; m[1] = v.y; m[2] = v.z; m[3] = v.w;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) m[i] = cm[IN_LDS ? 0 : (rt * C::HBL + (4 * k + i) % C::HBL) * NT + nt];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[rt][nt][4 * k + i] *= m[i];
                        amax[4 * k / C::HBL] = fmaxf(amax[4 * k / C::HBL], fabsf(acc[rt][nt][4 * k + i]));
                    }
                }
        float inv[C::T];
        bool bounded[C::T], all_bounded = true;
#pragma unroll
        for (int t = 0; t < C::T; ++t) {
            const int row = tile * TOK + (HB == 8 ? 2 * t + g : HB == 16 ? g : 0);
            float delta;
            if (step != nullptr) {
                delta = step[(size_t)min(row, rows - 1) * step_stride];
                inv[t] = delta >= kMinStep ? 1.0f / delta : 0.0f;
            } else {
                const float m = HB >= 32 ? max_over_64_lanes(amax[t]) : max_over_32_lanes(amax[t]);
                const bool live = m >= qmax * kMinStep;
                delta = live ? m / qmax : 0.0f;
                inv[t] = live ? qmax / m : 0.0f;
            }
            if (c == 0 && (HB < 32 || g == 0) && row < rows) scale[row] = delta;
            // a step from the row's own maximum bounds the ratio (see rotate_rows_general_kernel); the general form is for the others
            bounded[t] = step == nullptr && inv[t] > 0.0f;
            all_bounded = all_bounded && bounded[t];
        }
        lanes_exchange_fence();         // the codes go where other lanes' inputs were read
        auto stage_codes = [&](auto code_of) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int t = r / C::HBL, k = r / 4;
                        const int segment = r % 4 + (HB == 8 ? 4 * (k & 1) : HB == 16 ? 4 * k : 4 * (k & 1) + 16 * (k >> 1) + 32 * rt);
                        uint8_t *const at = lds + code_lane + (HB == 8 ? 2 * t * CODE_PITCH : 0) + CODE_BYTES * (8 * segment * MM + 4 * nt);
                        const uint32_t code = code_of(acc[rt][nt][r], t);
                        if constexpr (WIDE) *reinterpret_cast<uint16_t *>(at) = (uint16_t)(code >> 16);
                        else *at = (uint8_t)code;
                    }
        };
        // code of a value whose row has no code range or a given step
        auto general_code = [&](float v, int t) { return min(q_hi, max(q_lo, (int)__builtin_rintf(v * inv[t]))); };
        const bool fast = __builtin_amdgcn_ballot_w64(!all_bounded) == 0;
        if constexpr (WIDE) {               // the upper half of a small whole float is the bf16 number
            if (fast) stage_codes([&](float v, int t) { return __float_as_uint(fmaf(v, inv[t], kRoundMagic) - kRoundMagic); });
            else stage_codes([&](float v, int t) { return __float_as_uint(bounded[t] ? fmaf(v, inv[t], kRoundMagic) - kRoundMagic : (float)general_code(v, t)); });
        } else {
            if (fast) stage_codes([&](float v, int t) { return __float_as_uint(fmaf(v, inv[t], kRoundMagic)); });
            else stage_codes([&](float v, int t) { return bounded[t] ? __float_as_uint(fmaf(v, inv[t], kRoundMagic)) : (uint32_t)general_code(v, t); });
        }
        if constexpr (BLOCK_FLUSH) __syncthreads();
        else lanes_exchange_fence();
        if constexpr (CB == 6) {
            constexpr int R = BLOCK_FLUSH ? WAVES : TOK, THREADS = BLOCK_FLUSH ? WAVES * 64 : 64, STRIDE = BLOCK_FLUSH ? C::WAVE_LDS : CODE_PITCH;
            const uint8_t *const codes0 = BLOCK_FLUSH ? smem : lds;
            const int row0 = BLOCK_FLUSH ? tile - wave_in_block : tile * TOK;
            uint8_t *const block = out + (size_t)(row0 / 128) * (K / 64) * 6144 + (size_t)(row0 % 128) * 48;
            for (int i = BLOCK_FLUSH ? (int)threadIdx.x : lane; i < K / 32 * R; i += THREADS) {          // 32 codes each: unit, row, half
                const int h = i & 1, r = (i >> 1) % R, unit = (i >> 1) / R;
                if (row0 + r >= rows) continue;
                const uint8_t *codes = codes0 + r * STRIDE + (64 * unit + 32 * h) * 2;
                typedef unsigned int v16u __attribute__((ext_vector_type(16)));
                v16u v;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const v4u w = reinterpret_cast<const v4u *>(codes)[d];
                    v[4 * d] = w[0]; v[4 * d + 1] = w[1]; v[4 * d + 2] = w[2]; v[4 * d + 3] = w[3];
                }
                e2m3_v6u blob;
                asm volatile("v_cvt_scalef32_pk32_fp6_bf16 %0, %1, 1.0" : "=&v"(blob) : "v"(v));      // early clobber: as in e2m3_blob
                uint8_t *u = block + (size_t)unit * 6144 + r * 48;
                *reinterpret_cast<uint4 *>(u + h * 16) = make_uint4(blob[0], blob[1], blob[2], blob[3]);
                *reinterpret_cast<uint2 *>(u + 32 + h * 8) = make_uint2(blob[4], blob[5]);
            }
        } else {
            constexpr int PER_ROW = CB == 4 ? K / 32 : K / 16;                                           // 16-byte pieces
            for (int i = lane; i < PER_ROW * TOK; i += 64) {
                const int r = i / PER_ROW, piece = i % PER_ROW, row = tile * TOK + r;
                if (row >= rows) continue;
                const uint8_t *codes = lds + r * CODE_PITCH + piece * (CB == 4 ? 32 : 16);
                *reinterpret_cast<uint4 *>(out + (size_t)row * (K * CB / 8) + 16 * piece) = CB == 4 ? packed_codes(codes) : *reinterpret_cast<const uint4 *>(codes);
            }
        }
        if constexpr (BLOCK_FLUSH) __syncthreads();
        else lanes_exchange_fence();    // the next tile is staged where other lanes' codes were read
    }
}

template <int MM, int HB>
static hipError_t launch_paley(const void *X, int rows, const int8_t *signs, const float *mul, uint8_t *out, float *scale,
                               const float *step, int step_stride, int form, float qmax, hipStream_t stream)
{
    using C = pal::Cfg<MM, HB>;
    const int tiles = (rows + C::TOK - 1) / C::TOK, blocks = std::min((tiles + C::WAVES - 1) / C::WAVES, 256 * C::BLOCKS_PER_CU);
    const uint16_t *x = reinterpret_cast<const uint16_t *>(X);
#define QVGGT_PALEY(CB_) rotate_quant_paley_kernel<MM, HB, CB_><<<blocks, C::WAVES * 64, 0, stream>>>(x, rows, signs, mul, out, scale, step, step_stride, qmax)
    if (form == 6) QVGGT_PALEY(6);
    else if (form == 4) QVGGT_PALEY(4);
    else QVGGT_PALEY(8);
#undef QVGGT_PALEY
    return hipGetLastError();
}

// From how many bf16 activation rows this kernel is the faster one.  A wave has 3072 to 8192 values of its own, the general kernel's a quarter of that or
// less, so that few rows are better off there (16 rows with 512 channels: K = 2560 11.2 us there, 12.7 here, 5120 11.1 / 15.6, 6144 12.2 / 17.4).  us
// there / here, the layer with 512 channels, E2M3 codes and in brackets int8 rows:
//    768   1374  9.1 /  9.4           4097 12.6 / 12.2 (14.7 / 14.7)    24000  34.2 /  31.0  (35.1 /  35.4)
//   1536   1374 11.8 / 11.2 (15.8 / 15.6)  4097 17.9 / 16.3 (21.2 / 20.0)    24000  53.6 /  42.2  (58.5 /  49.7)
//   3072     16 12.1 / 10.3 (13.7 / 11.9)  4097 33.6 / 27.4 (38.7 / 34.0)    24000 111.1 /  74.3 (117.3 /  84.2)
//   6144   2300 42.7 / 42.8 (51.9 / 53.3)  4097 65.2 / 49.7 (61.6 / 55.2)    24000 254.2 / 148.8 (248.9 / 170.3)
//   2560   1374 16.3 / 16.7 (25.0 / 25.6)  4097 26.5 / 23.4 (31.8 / 30.3)    24000  84.4 /  63.2  (92.3 /  75.6)
//   5120   2300 33.8 / 35.2 (47.8 / 48.0)  4097 49.7 / 41.4 (56.3 / 49.7)    24000 187.8 / 123.7 (219.7 / 141.1)
//   8192   2300 52.1 / 51.9 (61.7 / 62.1)  4097 81.5 / 70.3 (80.6 / 75.9)    24000 342.6 / 255.8 (373.9 / 266.2)   (there: rotate_rows_kernel)
// One rule for all forms, which hold the same codes.  Sizes that begin a round of tiles lose by it: 5000 x 2560 28.4 / 28.8 (33.6 / 35.1), int8 rows
// 10992 x 1536 34.0 / 35.6, 16384 x 768 27.0 / 27.8.  Not here: K = 1280 (16384 rows 26.9 / 25.0, with 2748 14.8 / 15.3 and as int8 rows behind up to
// 8192), and m = 28, whose fragments and rows leave room for one wave per SIMD (16384 x 3584 82 / 60, but 2748 31.8 / 32.5 and 16 13.6 / 15.6; 8192 x 1792
// 28.7 / 33.4; six waves of a block are slower still).
int paley_matrix_core_rows(int K)
{
    switch (K) {
        case 768: return 3000;
        case 1536: return 1000;
        case 3072: return 1;
        case 6144: return 2700;
        case 2560: return 2000;
        case 5120: return 2500;
        case 8192: return 2400;
        default: return INT_MAX;
    }
}

// bf16 rows of a size that paley_matrix_core_rows() has.  form: 4 packed nibbles, 8 int8 rows, 6 E2M3 blocks (dynamic steps).  mul: inv_smooth or
// nullptr (1 / sqrt(K)); qmax: largest code; step: given steps or nullptr.
hipError_t run_rotate_quant_paley(const void *X, int rows, int K, const int8_t *signs, const float *mul, uint8_t *out, float *scale,
                                  const float *step, int step_stride, int form, float qmax, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
#define QVGGT_CASE(KK, MM, HB) \
    case KK: return launch_paley<MM, HB>(X, rows, signs, mul, out, scale, step, step_stride, form, qmax, stream);
    switch (K) {
        QVGGT_CASE(768, 12, 8)
        QVGGT_CASE(1536, 12, 16)
        QVGGT_CASE(3072, 12, 32)
        QVGGT_CASE(6144, 12, 64)
        QVGGT_CASE(2560, 20, 16)
        QVGGT_CASE(5120, 20, 32)
        QVGGT_CASE(8192, 16, 64)
        default: return hipErrorInvalidValue;
    }
#undef QVGGT_CASE
}

}  // namespace qvggt
