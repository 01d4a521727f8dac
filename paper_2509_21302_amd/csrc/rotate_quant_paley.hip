// Kernel 1 on the matrix cores for bf16 activation rows of K = 2^n * m values, m = 12 or 20 (a Paley factor; not K = 1280), and of K = 8192 (H_16 in its
// place).  fp32 rows, weights, the column statistic and the other sizes are in rotate_quant_general.hip, resp. rotate_quant.hip.
//
// H_K = H_{K / S} (x) (H_8 (x) H_m), S = 8 m = 96, 160 or 128.  A row is a (K / S) x S matrix of segments; its product with the right factor is taken
// on the matrix cores: the inputs and the +-1 entries are exact bf16 operands, the sums accumulate in fp32, and S is whole in 32-column
// tiles where m itself would leave lanes idle.  The left factor is 3 to 6 butterfly stages between the accumulator registers, as in
// rotate_quant_mfma.hip, whose order of MFMA rows this kernel has.
//
// Order of the contraction: a k-step of 16 is four values of b (4 q ..) for four values of the segment's three-bit index a (bit 2: the step,
// bit 1: the lane half, bit 0: the operand's two pieces of 8 bytes); a column tile is four outputs b' (4 nt ..) for all eight a'.  The operand
// of the +-1 entries then depends on the step only through q, and through the sign of bit 2 of a' (one xor): m^2 / 16 fragments instead of twice as many.
//
// Two kernels, of which whole_tile_rows() chooses by the number of rows.  rotate_quant_paley_columns_kernel: a block takes a tile, each of its m / 4 waves a
// column tile of it, with the m / 4 fragments of that in registers and the multipliers in LDS.  rotate_quant_paley_kernel: a wave takes whole tiles, for
// which all fragments are in registers for m = 12 (36; at K = 6144 there is no room), in LDS otherwise (25 KiB), and a tile's inputs are read from LDS
// once instead of m / 4 times.  A value goes through the same operations in the same order in both: a row's codes and step do not depend on how
// many rows come with it.
//
// Codes are in natural order (element e at position e).  A lane's results are one column of all segments; its codes go to LDS one by one, where the row's
// input was, and leave from there in whole units (E2M3: staged as bf16 numbers, which a conversion takes 32 at a time; converting staged bytes
// took 5 vector instructions a code instead of 2) or 16-byte pieces of a row.
//
// Whole tiles are bound by the vector ALU (12 to 14 instructions a value; busy 47 % of the clocks at 24000 x 3072 and x 5120) up to K = 1536 and by it and
// memory beyond: 16384 rows to E2M3, us of the general kernel / this one, K = 768 18.0 / 14.8 (2.3 TB/s), 1536 29.5 / 23.9, 3072 69.0 / 36.1 (3.8 TB/s),
// 6144 148 / 82, 2560 51.9 / 32.6, 5120 110 / 66.8.  Two waves per SIMD, for which some variants spill registers: 9 to 11 of 256 at K = 6144, up to 4 at 1536,
// 3072 and 5120; m = 20 and K = 6144 with one wave per SIMD took 41.0, 76.7 and 87.1.
// Column tiles are bound by latency, three barriers a tile with 1.5 to 1.7 waves per SIMD: 7000 x 5120 39 us (3.2 TB/s), vector ALU busy 40 %, LDS 23 %;
// 10992 x 768 10.3 us (2.3 TB/s), 29 % and 10 %; only at K = 8192 is LDS near half (16384 rows 129 us, 47 %, more than half of it bank conflicts).  us of a layer
// with 512 channels, the general kernel (K = 8192: rotate_rows_kernel) in front / this one, 16 rows and 4097: K = 768 6.9 / 6.9 and 12.7 / 11.8, 1536 8.4 /
// 7.2 and 18.8 / 16.8, 3072 12.1 / 8.1 and 34.4 / 25.7, 6144 12.0 / 11.1 and 65.8 / 43.0, 2560 11.2 / 8.3 and 27.3 / 25.0, 5120 10.9 / 9.8 and 50.5 / 39.4,
// 8192 14.3 / 12.7 and 82.2 / 56.6; as packed or int8 rows up to 1024 rows of 768 values take 0.1 to 0.3 longer than there (7.0 / 7.2, 8.6 / 8.8).
#include "paley.h"
#include "qvggt_common.h"
#include "rotate_rows.h"

#include <algorithm>
#include <climits>
#include <type_traits>

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
    static constexpr int WAVES = SHARED ? 8 : 4;
    static constexpr int BLOCKS_PER_CU = SHARED ? 1 : 2, WAVES_PER_SIMD = WAVES * BLOCKS_PER_CU / 4;
    static constexpr bool TABLES_IN_LDS = MM != 12 || SHARED;         // the +-1 fragments and the multipliers
    static constexpr int FRAGMENTS_AT = WAVES * WAVE_LDS, MULTIPLIERS_AT = FRAGMENTS_AT + (TABLES_IN_LDS ? NT * NT * 1024 : 0);
    static constexpr int LDS_BYTES = MULTIPLIERS_AT + (TABLES_IN_LDS ? K * 4 : 0);
    static constexpr bool WHOLE_TILES = MM != 16;                     // eight waves' rows of 8192 values are 136 KiB and the tables 48
    // Blocks of the columns kernel; as measured (a layer with 512 channels, 5 / 4 / 3 / 2 blocks): 768 4097 rows 11.8 / 11.8 / 12.5 / 13.5 us, 2560 2048 rows
    // - / 18.6 / 16.5 / 15.6, 5120 4097 rows - / 47.9 / 45.7 / 39.4, 8192 E2M3 4097 rows - / 59.1 / 65.7 / 56.6; 6144 differs with the last round, 4 at 8192
    // rows 62.2, 3 63.0, 2 73.1, at 10992 90.6 / 85.1 / 95.8
    static constexpr int COLUMN_BLOCKS_PER_CU = MM != 12 ? 2 : RT == 1 ? 5 : 4;
    static_assert(!WHOLE_TILES || LDS_BYTES * BLOCKS_PER_CU <= 160 * 1024, "the blocks of a compute unit share its LDS");
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

// sign masks of eight values, from their +-1 bytes
__device__ inline uint4 sign_masks(uint2 s)
{
    auto two = [](uint32_t w) { return ((w & 0x80u) << 8) | ((w & 0x8000u) << 16); };
    return make_uint4(two(s.x), two(s.x >> 16), two(s.y), two(s.y >> 16));
}

// The +-1 entries of k-step q with bit 2 of a = 0, column tile nt: element i (piece i / 4, value 4 q + i % 4) of the lane's column
template <int MM>
__device__ inline v4u fragment(int q, int nt, int lane)
{
    constexpr NegRows<MM> neg;
    const int g = lane >> 5, a_out = (lane & 31) >> 2, bit = 4 * nt + (lane & 3);
    const uint32_t one[2] = {0x3F803F80u ^ ((__popc((2 * g) & a_out) & 1) ? 0x80008000u : 0u), 0x3F803F80u ^ ((__popc((2 * g + 1) & a_out) & 1) ? 0x80008000u : 0u)};
    v4u w;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int b = 4 * q + 2 * (d & 1);
        w[d] = one[d >> 1] ^ ((neg.row[b] >> bit & 1u) << 15) ^ ((neg.row[b + 1] >> bit) << 31);
    }
    return w;
}

// The lane's inputs of a k-step, at p in a staged segment
template <int MM>
__device__ inline v8bf inputs(const uint8_t *p)
{
    const v2u p0 = *reinterpret_cast<const v2u *>(p), p1 = *reinterpret_cast<const v2u *>(p + 2 * MM);
    return __builtin_bit_cast(v8bf, (v4u){p0[0], p0[1], p1[0], p1[1]});
}

// H_{K / S} over the segments of a column tile: register bits 0, 1, 2, (3), the lane half, the row tile
template <int HB, int RT>
__device__ inline void segment_butterflies(v16f (&acc)[RT])
{
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int s = 0; s < (HB >= 16 ? 4 : 3); ++s) {
            const int h = 1 << s;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r & h) == 0) {
                    const float a = acc[rt][r], d = acc[rt][r + h];
                    acc[rt][r] = a + d;
                    acc[rt][r + h] = a - d;
                }
        }
        if constexpr (HB >= 32) {
            // hb bit 4 is the lane half: halves are swapped between registers r and r + 8 (register bit 3 means hb4 then, the lane half hb3)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[rt][r]), __float_as_uint(acc[rt][r + 8]), false, false);
                const float a = __uint_as_float(sw[0]), d = __uint_as_float(sw[1]);
                acc[rt][r] = a + d;
                acc[rt][r + 8] = a - d;
            }
        }
    }
    if constexpr (RT == 2) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float a = acc[0][r], d = acc[RT - 1][r];
            acc[0][r] = a + d;
            acc[RT - 1][r] = a - d;
        }
    }
}

// Segment (of its token) of register r of row tile rt, but for the lane half's share where HB >= 32
template <int HB>
constexpr int segment_of_register(int rt, int r)
{
    const int k = r / 4;
    return r % 4 + (HB == 8 ? 4 * (k & 1) : HB == 16 ? 4 * k : 4 * (k & 1) + 16 * (k >> 1) + 32 * rt);
}

// A row's step: given, or from the row's largest value
struct RowStep {
    float delta, inv;
    bool bounded;
    __device__ RowStep(float largest, const float *given, float qmax)
    {
        if (given != nullptr) {
            delta = *given;
            inv = delta >= kMinStep ? 1.0f / delta : 0.0f;
        } else {
            const bool live = largest >= qmax * kMinStep;
            delta = live ? largest / qmax : 0.0f;
            inv = live ? qmax / largest : 0.0f;
        }
        // a step from the row's own maximum bounds the ratio (see rotate_rows_general_kernel); the general form is for the others
        bounded = given == nullptr && inv > 0.0f;
    }
};

// What is staged of a value: the upper half of a bf16 number (WIDE: that of a small whole float is one), or a byte.  FAST: the row's step is bounded
template <bool WIDE, bool FAST>
__device__ inline void stage_code(uint8_t *at, float v, float inv, bool bounded, int q_lo, int q_hi)
{
    // a value whose row has no code range, or a given step
    auto general = [&]() { return min(q_hi, max(q_lo, (int)__builtin_rintf(v * inv))); };
    const float rounded = fmaf(v, inv, kRoundMagic);
    if constexpr (WIDE) *reinterpret_cast<uint16_t *>(at) = (uint16_t)(__float_as_uint(FAST || bounded ? rounded - kRoundMagic : (float)general()) >> 16);
    else *at = (uint8_t)(FAST || bounded ? __float_as_uint(rounded) : (uint32_t)general());
}

// THREADS threads write the codes of rows row0 .. row0 + R - 1, as far as they exist, staged CODE_PITCH bytes from row to row: E2M3 blocks (CB = 6, from bf16
// numbers), or rows of nibbles or bytes
template <int K, int CB, int R, int THREADS, int CODE_PITCH>
__device__ inline void write_codes(const uint8_t *staged, int row0, int rows, uint8_t *out, int thread)
{
    if constexpr (CB == 6) {
        uint8_t *const block = out + (size_t)(row0 / 128) * (K / 64) * 6144 + (size_t)(row0 % 128) * 48;
        for (int i = thread; i < K / 32 * R; i += THREADS) {          // 32 codes each: unit, row, half
            const int h = i & 1, r = (i >> 1) % R, unit = (i >> 1) / R;
            if (row0 + r >= rows) continue;
            const uint8_t *codes = staged + r * CODE_PITCH + (64 * unit + 32 * h) * 2;
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
        for (int i = thread; i < PER_ROW * R; i += THREADS) {
            const int r = i / PER_ROW, piece = i % PER_ROW, row = row0 + r;
            if (row >= rows) continue;
            const uint8_t *codes = staged + r * CODE_PITCH + piece * (CB == 4 ? 32 : 16);
            *reinterpret_cast<uint4 *>(out + (size_t)row * (K * CB / 8) + 16 * piece) = CB == 4 ? packed_codes(codes) : *reinterpret_cast<const uint4 *>(codes);
        }
    }
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
    v4u frag[IN_LDS ? 1 : NT * NT];
    if constexpr (IN_LDS) {
#pragma unroll
        for (int f = 0; f < NT * NT; ++f)
            if (f % WAVES == wave_in_block) *reinterpret_cast<v4u *>(fragments + f * 1024 + lane * 16) = fragment<MM>(f / NT, f % NT, lane);
    } else {
#pragma unroll
        for (int f = 0; f < NT * NT; ++f) frag[f] = fragment<MM>(f / NT, f % NT, lane);
    }
    uint4 sgn[C::SIGN_CLASSES];                                // load j: sign masks of class j % SIGN_CLASSES
#pragma unroll
    for (int q = 0; q < C::SIGN_CLASSES; ++q) sgn[q] = sign_masks(sb[q]);
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
            v.x ^= sgn[q].x; v.y ^= sgn[q].y; v.z ^= sgn[q].z; v.w ^= sgn[q].w;
            *reinterpret_cast<uint4 *>(lds + wr[j % NT] + j / NT * 16 * C::PITCH) = v;
        }
        lanes_exchange_fence();
        if (tile + nwaves < ntiles) load_tile(tile + nwaves);

        v16f acc[NT][RT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nt][rt][r] = 0.0f;
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
                    const v8bf a = inputs<MM>(lds + rd + rt * 32 * C::PITCH + hi * 8 * MM + 8 * q);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if (hi == 1 && rt == 0) b[nt] = b[nt] ^ flip;
                        acc[nt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(v8bf, b[nt]), acc[nt][rt], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) segment_butterflies<HB>(acc[nt]);
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
                        acc[nt][rt][4 * k + i] *= m[i];
                        amax[4 * k / C::HBL] = fmaxf(amax[4 * k / C::HBL], fabsf(acc[nt][rt][4 * k + i]));
                    }
                }
        float inv[C::T];
        bool bounded[C::T], all_bounded = true;
#pragma unroll
        for (int t = 0; t < C::T; ++t) {
            const int row = tile * TOK + (HB == 8 ? 2 * t + g : HB == 16 ? g : 0);
            float largest = 0.0f;
            if (step == nullptr) largest = HB >= 32 ? max_over_64_lanes(amax[t]) : max_over_32_lanes(amax[t]);
            const RowStep s(largest, step != nullptr ? step + (size_t)min(row, rows - 1) * step_stride : nullptr, qmax);
            if (c == 0 && (HB < 32 || g == 0) && row < rows) scale[row] = s.delta;
            inv[t] = s.inv;
            bounded[t] = s.bounded;
            all_bounded = all_bounded && s.bounded;
        }
        lanes_exchange_fence();         // the codes go where other lanes' inputs were read
        auto stage_codes = [&](auto fast_c) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int t = r / C::HBL;
                        uint8_t *const at = lds + code_lane + (HB == 8 ? 2 * t * CODE_PITCH : 0) + CODE_BYTES * (8 * segment_of_register<HB>(rt, r) * MM + 4 * nt);
                        stage_code<WIDE, decltype(fast_c)::value>(at, acc[nt][rt][r], inv[t], bounded[t], q_lo, q_hi);
                    }
        };
        if (__builtin_amdgcn_ballot_w64(!all_bounded) == 0) stage_codes(std::true_type{});
        else stage_codes(std::false_type{});
        if constexpr (BLOCK_FLUSH) __syncthreads();
        else lanes_exchange_fence();
        if constexpr (BLOCK_FLUSH) write_codes<K, CB, WAVES, WAVES * 64, C::WAVE_LDS>(smem, tile - wave_in_block, rows, out, (int)threadIdx.x);
        else write_codes<K, CB, TOK, 64, CODE_PITCH>(lds, tile * TOK, rows, out, lane);
        if constexpr (BLOCK_FLUSH) __syncthreads();
        else lanes_exchange_fence();    // the next tile is staged where other lanes' codes were read
    }
}

// A block takes a tile, each of its NT waves one column tile.
template <int MM, int HB, int CB>
__global__ __launch_bounds__((pal::Cfg<MM, HB>::NT * 64)) void rotate_quant_paley_columns_kernel(
    const uint16_t *__restrict__ X, int rows, const int8_t *__restrict__ signs, const float *__restrict__ mul,
    uint8_t *__restrict__ out, float *__restrict__ scale, const float *__restrict__ step, int step_stride, float qmax)
{
    using namespace pal;
    using C = Cfg<MM, HB>;
    constexpr int K = C::K, NT = C::NT, RT = C::RT, TOK = C::TOK, THREADS = NT * 64;
    constexpr bool WIDE = CB == 6;
    constexpr int CODE_BYTES = WIDE ? 2 : 1, CODE_PITCH = CODE_BYTES * K + 16;
    static_assert(TOK * CODE_PITCH <= C::WAVE_LDS, "a tile's codes fit its staging rows");
    constexpr int LOADS = 2 * RT, SIGN_CLASSES = HB <= 16 ? 1 : HB / 16;      // 16-byte loads per thread: 16 segments each, and the positions of a row that they have
    static_assert(THREADS == 16 * MM && LOADS % SIGN_CLASSES == 0, "a load of the block is 16 segments");
    __shared__ __attribute__((aligned(16))) uint8_t lds[C::WAVE_LDS];
    __shared__ float4 multipliers[K / 4];                      // in natural order
    __shared__ float largest_of[NT][4];
    const int tid = (int)threadIdx.x, lane = tid & 63, nt = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, g = lane >> 5, a_out = c >> 2, j_out = c & 3;
    const int ntiles = (rows + TOK - 1) / TOK;

    const size_t max_flat = (size_t)rows * K;
    uint4 G[LOADS];
    auto load_tile = [&](int t) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            size_t f = (size_t)t * (TOK * K) + (size_t)(8 * (THREADS * j + tid));
            if (f >= max_flat) f = max_flat - K + f % K;               // rows past the end: the last row again, not written
            const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(X + f));
            G[j] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    };
    int tile = (int)blockIdx.x;
    load_tile(tile);
    uint2 sb[SIGN_CLASSES];
#pragma unroll
    for (int q = 0; q < SIGN_CLASSES; ++q) sb[q] = signs != nullptr ? *reinterpret_cast<const uint2 *>(signs + 8 * (THREADS * q + tid) % K) : make_uint2(0u, 0u);
    static_assert(HB % 8 == 0, "whole pieces of four per thread");
    const float rs = 1.0f / sqrtf((float)K);
    float4 cm4[HB / 8];
#pragma unroll
    for (int i = 0; i < HB / 8; ++i) cm4[i] = mul != nullptr ? reinterpret_cast<const float4 *>(mul)[THREADS * i + tid] : make_float4(rs, rs, rs, rs);
    v4u frag[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) frag[q] = fragment<MM>(q, nt, lane);
    uint4 sgn[SIGN_CLASSES];
#pragma unroll
    for (int q = 0; q < SIGN_CLASSES; ++q) sgn[q] = sign_masks(sb[q]);
#pragma unroll
    for (int i = 0; i < HB / 8; ++i) multipliers[THREADS * i + tid] = cm4[i];
    const uint32_t flip = (c & 16) ? 0x80008000u : 0u;
    uint8_t *const wr = lds + tid / MM * C::PITCH + tid % MM * 16;
    const uint8_t *const rd = lds + segment_of_row<HB>(c) * C::PITCH + g * 4 * MM;
    const float *const cm = reinterpret_cast<const float *>(multipliers) + (HB >= 32 ? 64 * MM * g : 0) + a_out * MM + 4 * nt + j_out;
    uint8_t *const code_lane = lds + CODE_BYTES * (a_out * MM + 4 * nt + j_out) + g * (HB >= 32 ? CODE_BYTES * 64 * MM : CODE_PITCH);
    const int q_hi = (int)qmax, q_lo = -q_hi - 1;

    for (;;) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            uint4 v = G[j];
            const uint4 m = sgn[j % SIGN_CLASSES];
            v.x ^= m.x; v.y ^= m.y; v.z ^= m.z; v.w ^= m.w;
            *reinterpret_cast<uint4 *>(wr + j * 16 * C::PITCH) = v;
        }
        __syncthreads();
        const int next = tile + (int)gridDim.x;
        if (next < ntiles) load_tile(next);

        v16f acc[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rt][r] = 0.0f;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const v4u b = hi == 0 ? frag[q] : frag[q] ^ flip;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(inputs<MM>(rd + rt * 32 * C::PITCH + hi * 8 * MM + 8 * q), __builtin_bit_cast(v8bf, b), acc[rt], 0, 0, 0);
            }
        }
        segment_butterflies<HB>(acc);
        float amax[C::T];
#pragma unroll
        for (int t = 0; t < C::T; ++t) amax[t] = 0.0f;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[rt][r] *= cm[8 * MM * segment_of_register<HB>(rt, r)];
                amax[r / C::HBL] = fmaxf(amax[r / C::HBL], fabsf(acc[rt][r]));
            }
        auto token_of = [&](int t) { return HB == 8 ? 2 * t + g : HB == 16 ? g : 0; };
        if (step == nullptr) {
#pragma unroll
            for (int t = 0; t < C::T; ++t) {
                const float m = HB >= 32 ? max_over_64_lanes(amax[t]) : max_over_32_lanes(amax[t]);
                if (c == 0) largest_of[nt][token_of(t)] = m;
            }
        }
        __syncthreads();                // and the codes go where inputs were read
        float inv[C::T];
        bool bounded[C::T], all_bounded = true;
#pragma unroll
        for (int t = 0; t < C::T; ++t) {
            const int row = tile * TOK + token_of(t);
            float largest = 0.0f;
            if (step == nullptr) {
#pragma unroll
                for (int w = 0; w < NT; ++w) largest = fmaxf(largest, largest_of[w][token_of(t)]);
            }
            const RowStep s(largest, step != nullptr ? step + (size_t)min(row, rows - 1) * step_stride : nullptr, qmax);
            if (nt == 0 && c == 0 && (HB < 32 || g == 0) && row < rows) scale[row] = s.delta;
            inv[t] = s.inv;
            bounded[t] = s.bounded;
            all_bounded = all_bounded && s.bounded;
        }
        auto stage_codes = [&](auto fast_c) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int t = r / C::HBL;
                    uint8_t *const at = code_lane + (HB == 8 ? 2 * t * CODE_PITCH : 0) + CODE_BYTES * 8 * segment_of_register<HB>(rt, r) * MM;
                    stage_code<WIDE, decltype(fast_c)::value>(at, acc[rt][r], inv[t], bounded[t], q_lo, q_hi);
                }
        };
        if (__builtin_amdgcn_ballot_w64(!all_bounded) == 0) stage_codes(std::true_type{});
        else stage_codes(std::false_type{});
        __syncthreads();
        write_codes<K, CB, TOK, THREADS, CODE_PITCH>(lds, tile * TOK, rows, out, tid);
        if (next >= ntiles) return;     // the whole block
        tile = next;
        __syncthreads();                // the next tile is staged where codes were read
    }
}

// From how many rows a wave with whole tiles is the faster one.  us of a layer with 512 channels, columns kernel / whole tiles, E2M3 codes and in brackets
// int8 rows:
//    768   4097 11.8 / 12.2 (14.4 / 15.0)  13000  21.3 /  21.3 (24.1 /  24.8)   34350  39.8 /  38.7 (50.9 /  48.6)
//   1536   4097 16.8 / 17.2 (20.1 / 20.9)  20000  40.6 /  40.5 (45.7 /  45.8)   34350  62.0 /  57.3 (75.3 /  72.8)
//   3072   1374 15.1 / 16.7 (25.0 / 26.7)   7000  33.3 /  33.0 (39.3 /  39.2)   24000  86.5 /  78.3 (92.3 /  88.0)
//   6144   4097 43.0 / 49.0 (52.0 / 56.0)   8192  62.9 /  64.0 (71.9 /  73.8)   30000 227.3 / 186.0 (253.1 / 221.3)
//   2560   2048 15.6 / 18.0 (23.8 / 26.6)  10992  43.5 /  43.2 (51.3 /  53.3)   24000  79.1 /  68.3 (88.2 /  80.3)
//   5120   2048 24.7 / 25.5 (41.3 / 41.6)   7000  52.4 /  55.2 (61.3 /  64.6)    8192  61.1 /  56.6 (70.3 /  65.4)
// K = 6144 goes up and down with the rounds of either kernel (14500 rows 97.8 / 108.0, 20000 158.5 / 132.0).  K = 8192: whole tiles have room for one wave per
// SIMD and are the slower ones at all sizes (4097 rows 59 / 69, 16384 163 / 171).
// Not here: K = 1280 (16384 rows 26.9 us in the general kernel, 25.0 in whole tiles, but 2748 14.8 / 15.3), and m = 28, whose fragments and rows leave room for
// one wave of whole tiles per SIMD (16384 x 3584 82 / 60, but 2748 31.8 / 32.5 and 16 13.6 / 15.6; 8192 x 1792 28.7 / 33.4); neither was tried in columns.
static int whole_tile_rows(int K)
{
    switch (K) {
        case 768: return 13500;
        case 1536: return 20000;
        case 3072: return 7000;
        case 6144: return 9000;
        case 2560: return 11500;
        case 5120: return 7600;
        default: return INT_MAX;
    }
}

template <int MM, int HB>
static hipError_t launch_paley(const void *X, int rows, const int8_t *signs, const float *mul, uint8_t *out, float *scale,
                               const float *step, int step_stride, int form, float qmax, hipStream_t stream)
{
    using C = pal::Cfg<MM, HB>;
    const int tiles = (rows + C::TOK - 1) / C::TOK;
    const uint16_t *x = reinterpret_cast<const uint16_t *>(X);
    const auto launch = [&](auto kernel, int blocks, int threads) {
        kernel<<<blocks, threads, 0, stream>>>(x, rows, signs, mul, out, scale, step, step_stride, qmax);
        return hipGetLastError();
    };
    if constexpr (C::WHOLE_TILES) {
        if (rows >= whole_tile_rows(C::K)) {
            const int blocks = std::min((tiles + C::WAVES - 1) / C::WAVES, 256 * C::BLOCKS_PER_CU);
            return launch(form == 6 ? rotate_quant_paley_kernel<MM, HB, 6> : form == 4 ? rotate_quant_paley_kernel<MM, HB, 4> : rotate_quant_paley_kernel<MM, HB, 8>,
                          blocks, C::WAVES * 64);
        }
    }
    return launch(form == 6 ? rotate_quant_paley_columns_kernel<MM, HB, 6> : form == 4 ? rotate_quant_paley_columns_kernel<MM, HB, 4> : rotate_quant_paley_columns_kernel<MM, HB, 8>,
                  std::min(tiles, 256 * C::COLUMN_BLOCKS_PER_CU), C::NT * 64);
}

// bf16 rows of a size that paley_size() has.  form: 4 packed nibbles, 8 int8 rows, 6 E2M3 blocks (dynamic steps).  mul: inv_smooth or
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
