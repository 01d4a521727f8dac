// Which tile configuration of the two GEMMs (int8 instructions, E2M3) runs where: a function of the problem's sizes alone, on the host and
// without HIP, so that it can be looked at without a GPU.
#pragma once

#include <algorithm>
#include <cmath>

namespace qvggt {

// Which 256 x 256 tiles of E2M3 codes and of int8 blocks are on the 16 x 16 matrix instructions (gemm_tiles256.h) and which on the 32 x 32 ones (gemm_e2m3.hip,
// gemm_w4a4.hip).  The 16 x 16 ones take less power, which bounds whole rounds of the chip, but about 2 us more of a launch's first and last tiles, and where K is short
// more of every tile.  t: tiles per compute unit.  Time of 32 x 32 over that of 16 x 16, the means of 3 to 6 problems of a bin (650 in all):
//              t < 0.6   0.6 - 0.8   0.8 - 0.95   0.95 - 1   1 - 2   2 - 5   more
//   int8  768   0.91       0.94        0.93         0.95      1.01    1.01    1.02
//        1280   0.98       0.96        0.98                   1.00    1.03    1.05
//        2048   0.97       0.99        1.06         1.02      1.03    1.04    1.04
//        3072   0.99       1.03                     1.03      1.06    1.06    1.06
//        8192   0.98       1.06        1.10         1.05      1.06    1.07    1.10
//   E2M3  768              0.93        0.96         0.96      0.98    1.00    0.98
//        1280              0.94        0.97         1.01      1.00    1.01    1.02
//        2048              0.97        0.97         0.99      1.01    1.02    1.01
//        3072              1.00        1.01         1.00      1.03    1.03    1.04
//        8192              1.06        1.05         1.02      1.06    1.04    1.05
// Affine E2M3 codes as plain ones.  us: int8 blocks 11660 x 768 -> 736 13.0 / 15.2, 12870 x 1024 -> 768 15.2 / 17.5, 24705 x 8192 -> 1056 193 / 175; E2M3
// 25447 x 1280 -> 480 16.8 / 18.0, 16381 x 128 -> 1024 10.7 / 12.0, 32976 x 4096 -> 2048 144 / 137.
constexpr int TILES256_LEAST_K = 768;
constexpr double tiles256_per_unit(int M, int N) { return (double)((M + 255) / 256) * ((N + 255) / 256) / 256.0; }
constexpr bool e2m3_tiles256(int M, int N, int K)
{
    const double t = tiles256_per_unit(M, N);
    return t > 1.0 ? K >= 1280 : K * (t - 0.3) >= 1400.0;
}
constexpr bool i8b_tiles256(int M, int N, int K)
{
    const double t = tiles256_per_unit(M, N);
    return t > 1.0 ? K >= TILES256_LEAST_K : K * (t - 0.5) >= 640.0;
}

struct GemmPlan {
    enum Shape { kBig, kSmall, kDeep, kBigThenDeep } shape;
    int rows_main;      // kBigThenDeep: the token rows (whole 256-row tiles) that go to the big tiles
};

// The plan that the model below prices lowest, in microseconds.  Rows are independent, so token rows can be divided between configurations.
//   big    256 x 256 tiles, one per compute unit: whole rounds of 256, a last one that is mostly empty costs as much as a full one.
//   small  128 x 128 tiles, two blocks per compute unit, one's epilogue under the other's K loop: while all compute units have two, the cost
//          follows the number of tiles (packed codes, 10992 x 768 -> 3072: 2064 tiles are 4.03 rounds of 512, not 5), and a tile costs 1.0 of a
//          quarter of a big one at K = 128, 1.14 at 1024, 1.4 at 4096 (int8 codes: 1.2 and 1.75), the LDS traffic per MFMA being twice as
//          much.  The tiles left after whole rounds run alone on their compute units: as a share of a round they cost at least
//          LAST_ROUND however few they are (int8 blocks at K = 2048: 484 tiles 21 us, 540 tiles 34, 836 tiles 36; at K = 4096: 475 tiles 35,
//          519 tiles 62, 830 tiles 66).
//   deep   128 x 128 tiles, one block per compute unit with an eight-stage ring: for at most 256 of them, where a tile's time is its chain of
//          transfers (int8 codes, 1374 x 4096 -> 1024: 31 -> 16 us; packed codes 22 -> 18 us for 700 x 4096 -> 4096).  Filling the longer ring
//          costs 0.2 to 0.4 us, which the chain has to be long enough to pay back.  Packed codes, small / deep: 509 rows -> 1024 (32 tiles) 7.4 /
//          7.7 us at K = 1024, 10.3 / 10.5 at 2048, 13.2 / 13.2 at 3072, 16.1 / 16.2 at 4096, 22.5 / 22.0 at 6144; with more tiles two
//          small ones meet on a compute unit: 953 rows -> 2896 (184 tiles) 20.1 / 16.8 at 3584, 1021 -> 2048 (128) 21.4 / 17.4 at 4096.
//          Affine codes, whose scale area is larger, gain 1 to 2 % at K = 1024 and 4 % at 4096.  int8 codes: 509 rows -> 1024 5.9 / 6.1
//          at K = 512, 6.8 / 6.7 at 768 (but 2045 rows -> 2048 8.4 / 8.7), 7.6 / 7.3 at 1024, 10.5 / 9.8 at 2048.
//   tail   the token rows that fill whole big rounds in big tiles, the rest in deep ones, in one launch (us, big / small / tail): packed codes
//          17354 x 4096 -> 1184 87 / 89 / 80, 113324 x 768 -> 672 86 / 81 / 72; int8 rows 34003 x 2048 -> 480 53 / 53 / 43.
//          Few deep tiles after a whole round of them cost 0.6 of one (affine codes, 4298 x 3584 -> 4864, 304 of them: 82 / 87 / 77).
// Measured (us, big / small / tail): packed codes 10992 x 768 -> 3072 42.6 / 33.6 / 38.1, 32976 x 256 -> 3072 56 / 50 / 55,
// 32976 x 1024 -> 1024 50 / 40 / 45, 32976 x 4096 -> 1024 137 / 130 / 113; int8 blocks 32976 x 4096 -> 1024 140 / 156 / 118,
// 20000 x 4096 -> 1024 89 / 92 / 71; just past one round of small tiles (big / small) int8 rows 9591 x 4096 -> 896 43 / 66,
// int8 blocks 22039 x 4096 -> 304 45 / 62, 2247 x 2048 -> 4256 27 / 36, packed codes 39144 x 5120 -> 160 48 / 55.  These and the prices of int8 blocks' big tiles are of
// the 32x32x32 instruction; where i8b_tiles256 has them on the 16x16x64 one they take 2 to 10 % less.
// affine and dump: affine activation codes, the accumulator dump (their two tile loops do not fit the registers together: two launches).
inline GemmPlan int8_instruction_gemm_plan(int M, int N, int K, int code_bits, bool affine, bool dump, double *cost = nullptr)
{
    auto tiles = [&](int rows, int size) { return (double)((rows + size - 1) / size) * ((N + size - 1) / size); };
    auto rounds = [](double t) { return std::ceil(t / 256.0); };
    const bool packed = code_bits == 4;
    const double k = K / 1024.0;
    const double big_round = 5.0 + (packed ? 11.0 : 12.0) * k, deep_round = 7.0 + 3.7 * k;
    const double small_share = 0.50 + (packed ? 0.055 : 0.095) * k;          // of a big round, for 512 small tiles
    const double LAST_ROUND = packed ? 0.3 : 0.5;
    const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256, ktiles = K * code_bits / (8 * 64);

    const double small_tiles = tiles(M, 128);
    const bool long_chain = !packed ? ktiles >= 16 : affine ? ktiles >= 8 : ktiles >= 28 && ktiles + small_tiles / 8.0 >= 40.0;
    if (small_tiles <= 256.0 && long_chain) {
        if (cost != nullptr) *cost = deep_round;
        return {GemmPlan::kDeep, 0};
    }
    const double big_cost = rounds(tiles(M, 256)) * big_round;
    const double small_rounds = small_tiles / 512.0, whole = std::floor(small_rounds), rest = small_rounds - whole;
    const double small_cost = (whole + (whole > 0.0 && rest > 0.0 ? std::max(rest, LAST_ROUND) : rest)) * small_share * big_round + 3.0;
    // whole tile rows that fit into the full rounds
    const int main_tile_rows = (int)std::min<double>(tiles_m, std::floor(tiles(M, 256) / 256.0) * 256.0 / tiles_n);
    if (main_tile_rows > 0 && main_tile_rows < tiles_m && ktiles >= 4) {        // the eight-stage ring needs three, and with few is filled with re-reads
        const int rows_main = main_tile_rows * 256;
        const double deep_rounds = tiles(M - rows_main, 128) / 256.0, deep_whole = std::floor(deep_rounds), deep_rest = deep_rounds - deep_whole;
        const double tail_cost = rounds((double)main_tile_rows * tiles_n) * big_round + (affine || dump ? 3.0 : 0.0) +
                                 (deep_whole + (deep_rest == 0.0 ? 0.0 : deep_whole > 0.0 ? std::max(deep_rest, 0.6) : 1.0)) * deep_round;
        if (tail_cost < std::min(big_cost, small_cost)) {
            if (cost != nullptr) *cost = tail_cost;
            return {GemmPlan::kBigThenDeep, rows_main};
        }
    }
    if (cost != nullptr) *cost = std::min(small_cost, big_cost);
    return {small_cost < big_cost ? GemmPlan::kSmall : GemmPlan::kBig, 0};
}

// Few tiles of the int8-instruction GEMM: the tokens x channels of w4a4_gemm_few_kernel, where it is faster than the plan above, or none.  Both
// sides in microseconds (k = K / 1024), fitted to 400 random problems of 16 to 4200 rows measured in every shape: the plan, for at most 256 tiles of
// 128 x 128, within 5 % of its time (rms), the three shapes, priced 4 % above what they took, within 4 to 9 %.  The choice is 1.42 times faster than
// the plan alone on geometric average, 3 % slower at worst.  us, plan / 64 x 64 / 32 x 64 / 32 x 32: int8 blocks 40 x 4096 -> 944 15.9 / 11.2 / 9.0 /
// 7.2, 424 x 2048 -> 4096 11.6 / 12.2 / 15.3 / 19.9, 533 x 1024 -> 1184 8.0 / 6.3 / 6.6 / 7.4; packed codes 23 x 4096 -> 1024 16.7 / 9.6 / 8.7 / 6.8; int8
// rows, whose fragments come in 32-byte pieces, 434 x 2048 -> 1024 10.7 / 11.3 / 9.3 / 11.3.
enum class FewTiles { kNone, k64, k32x64, k32 };
inline FewTiles int8_instruction_few_tiles(int M, int N, int K, int code_bits, bool blocks)
{
    auto tiles = [&](int m, int n) { return (double)((M + m - 1) / m) * ((N + n - 1) / n) / 256.0; };        // per compute unit
    const double k = K / 1024.0, t = tiles(128, 128);
    if (t > 1.0) return FewTiles::kNone;
    const bool packed = code_bits == 4;
    double best = packed ? 5.3 + 2.75 * k + t * (1.4 + 0.5 * k) : 5.1 + 2.6 * k + t * (1.2 + 1.1 * k);
    FewTiles shape = FewTiles::kNone;
    auto offer = [&](FewTiles s, double per_unit, double c0, double c1, double c2, double c3) {
        const double cost = 1.04 * (c0 + c1 * k + (std::ceil(per_unit) - 1.0) * (c2 + c3 * k));
        if (cost < best) { best = cost; shape = s; }
    };
    const double t64 = tiles(64, 64), t32x64 = tiles(32, 64), t32 = tiles(32, 32);
    if (packed) {
        offer(FewTiles::k64, t64, 5.0, 1.6, 1.55, 1.6);
        offer(FewTiles::k32x64, t32x64, 4.4, 1.2, 0.75, 1.2);
        offer(FewTiles::k32, t32, 4.85, 0.7, 1.4, 0.65);
    } else if (blocks) {
        offer(FewTiles::k64, t64, 4.25, 1.75, 0.6, 2.0);
        offer(FewTiles::k32x64, t32x64, 3.9, 1.25, 0.1, 1.5);
        offer(FewTiles::k32, t32, 4.0, 0.8, 0.5, 0.9);
    } else {
        offer(FewTiles::k64, t64, 4.65, 3.0, 0.85, 3.8);
        offer(FewTiles::k32x64, t32x64, 4.25, 2.35, 0.35, 2.65);
        offer(FewTiles::k32, t32, 4.4, 1.45, 0.5, 1.65);
    }
    return shape;
}

// Which tile shape of the E2M3 GEMM runs where.
struct E2m3Plan {
    enum Shape { k256, k192, k128, k64, k32x64, k32 } shape;
    int rows_main;      // token rows of `shape`: all of them, or whole 256-row tiles that fill whole rounds
    Shape rest;         // what takes the others, in a second launch
};

// Rows of Y that are whole 128-byte lines (N a multiple of 64) go past the caches.  Others are written in pieces of lines, which the memory
// takes badly one by one: while Y fits half the memory-side cache (256 MB; the rows of X go through it too), the 256- and 192-row tiles leave them
// there to be put together.  us at
// K = 1024, past the caches / through them, 256-row tiles: 2000 x 3056 (12 MB) 13.5 / 14.5, 4000 (24) 19.9 / 16.7, 10992 (67) 54 / 41, 34000 (208)
// 121 / 96, 50000 (306) 169 / 163, 192-row tiles 159 / 176.  The 128-row tiles, two blocks to a compute unit, do not gain (35.0 / 33.8, 91 / 90,
// 136 / 191), nor do whole lines (10992 x 4096 40.5 / 43.9, 1374 x 3072 12.6 / 13.8).
constexpr double kCachedY = 130e6;       // bytes
inline bool e2m3_streams_y(int M, int N)
{
    const double bytes = 2.0 * M * N;
    return N % 64 == 0 || bytes < 20e6 || bytes > kCachedY;
}

// Which tiles of an XCD's range are neighbours: those of one row of tokens, unless the weights are the larger operand and more than its L2 of
// 4 MiB holds with anything else.  Then those of one column: the XCD reads its share of the weights once and all tokens, instead of all
// weights.  us at K = 4096, channels first / tokens first: 85 x 4096 -> 4096 9.3 / 6.2 (32 x 64 tiles), 374 -> 3072 16.0 / 11.7 (64 x 64),
// 1374 -> 4096 24.0 / 20.7 (128 x 128); 1374 x 1024 -> 3072, whose weights fit, 8.8 / 9.0.  128 x 128 tiles that have a compute unit each only at
// K = 4096: with shorter K it costs them (with kernel 1: 670 x 2048 -> 3072 14.5 / 15.1, 1000 -> 3328 15.0 / 15.8, 1374 -> 2624 15.4 / 16.6; with more
// tiles 1182 -> 3840 19.6 / 18.8, 1374 -> 3696 20.0 / 19.7).
constexpr bool e2m3_tokens_first(int tiles_m, int tiles_n, int N, int K)
{
    return tiles_m < tiles_n && (long long)N * K > (4 << 20);
}
constexpr bool e2m3_128_tokens_first(int tiles_m, int tiles_n, int N, int K)
{
    return e2m3_tokens_first(tiles_m, tiles_n, N, K) && (K >= 4096 || tiles_m * tiles_n > 256);
}

// The plan that this model prices lowest, in microseconds, fitted to 550 random problems of 16 to 137400 rows and all sizes of K that were
// measured in every shape on two cards (as graph nodes, codes of a normal distribution): within 3 to 7 % of the time (rms).  The last three shapes are
// priced 4 % above what they took, the 128s' last word where it is close.  Measured as calls run it, behind kernel 1 and with codes of heavy-tailed
// rows, on 1940 problems: the choice is 1 % slower than the best on geometric average.  The 128s' round is priced by those measurements where the rows of
// Y are whole lines and K >= 1024 (K = 512 and 768 take the same time by either price: 10992 x 768 -> 3072 39.6 in 192s, 40.0 in 128s); as the fit had it, 2.1 + 4.95 k, it put 256s and 192s where 128s are the faster: with kernel 1, 6715 x 1024 -> 3072 27.4 / 24.9,
// 12759 -> 3072 52.1 / 48.3, 13091 -> 4096 62.6 / 56.0, 26106 -> 2048 74.1 / 65.7, 50838 -> 1024 85.7 / 73.9.
//   256, 192   tokens x 256 channels per block, one per compute unit: whole rounds of 256 tiles, and the tiles themselves (power).  192 rows
//              where they waste less of the last round: with kernel 1, 21984 x 4096 -> 1024 112.8 us in 256s, 103.8 in 192s, 10992 -> 1024 57.7 /
//              53.9; the LDS traffic per MFMA is a sixth more: 97554 x 1024 -> 1024 122 / 131.
//   256 and a rest   32976 x 4096 -> 1024 (2.02 rounds of 256) 157.5 us in 256s, 151.9 in 192s, 142.1 as 32768 rows in 256s and 208 in 32s.
//   128        128 x 128, two blocks per compute unit: by number beyond the first block, at least 0.3 of a round for a last one, 0.7 where some
//              units have two blocks in it: 10992 x 1024 -> 2048 (2.69 rounds) 35.0 in 128s, 33.9 in 192s.
//   64, 32x64, 32   tokens x channels, K divided among the block's waves (e2m3_gemm_few_kernel): for problems whose 128 x 128 tiles would walk along
//              K alone on their compute units (64 x 4096 -> 1024 13.3 us in 128s, 7.5 / 6.1 / 5.2 in these; 500 x 4096 -> 1024 13.2, 7.6 / 6.4 / 7.6;
//              1000 x 1024 -> 1024 6.7, 5.0 / 5.0 / 6.1; 1374 x 1024 -> 3072 8.9, 11.2 / 11.3 / 15.4).
inline double e2m3_shape_cost(E2m3Plan::Shape shape, int M, int N, int K)
{
    auto tiles = [&](int m, int n) { return (double)((M + m - 1) / m) * ((N + n - 1) / n) / 256.0; };        // per compute unit
    const double k = K / 1024.0, pieces = N % 64 == 0 ? 0.0 : 2.0 * M * N > kCachedY ? 4.0 : 1.0;
    switch (shape) {
        case E2m3Plan::k256: {
            const double t = tiles(256, 256);
            return 5.3 - 0.7 * k + std::ceil(t) * (3.4 + 4.85 * k) + t * (1.6 + 2.1 * k + 1.2 * pieces);
        }
        case E2m3Plan::k192: {
            const double t = tiles(192, 256);
            return 5.2 - 0.65 * k + std::ceil(t) * (2.5 + 4.25 * k) + t * (1.55 + 1.4 * k + 0.7 * pieces);
        }
        case E2m3Plan::k128: {
            const double t = tiles(128, 128), rounds = t / 2.0, whole = std::floor(rounds), rest = rounds - whole;
            const bool in_calls = pieces == 0.0 && K >= 1024;
            const double priced = whole > 0.0 && rest > 0.0 ? whole + std::max(rest, in_calls && rest > 0.5 ? 0.7 : 0.3) : rounds;
            const double round = in_calls ? 1.5 + 5.05 * k : 2.1 + 4.95 * k;
            return 5.05 + 2.2 * k + std::min(t, 1.0) * (1.2 + 0.6 * k) + std::max(priced - 0.5, 0.0) * std::max(round, 3.4 + std::min(1.8 * pieces, 1.8));
        }
        case E2m3Plan::k64: return 4.85 + 0.93 * k + (std::ceil(tiles(64, 64)) - 1.0) * (0.95 + 1.1 * k);
        case E2m3Plan::k32x64: return 4.45 + 0.65 * k + (std::ceil(tiles(32, 64)) - 1.0) * (0.38 + 0.81 * k);
        case E2m3Plan::k32: return 4.8 + 0.37 * k + (std::ceil(tiles(32, 32)) - 1.0) * (0.38 + 0.52 * k);
    }
    return 0.0;
}

inline E2m3Plan e2m3_gemm_plan(int M, int N, int K, double *cost = nullptr)
{
    auto cheapest = [&](int rows, double &cost) {
        E2m3Plan::Shape best = E2m3Plan::k256;
        cost = e2m3_shape_cost(best, rows, N, K);
        for (E2m3Plan::Shape s : {E2m3Plan::k192, E2m3Plan::k128, E2m3Plan::k64, E2m3Plan::k32x64, E2m3Plan::k32}) {
            const double c = e2m3_shape_cost(s, rows, N, K);
            if (c < cost) { cost = c; best = s; }
        }
        return best;
    };
    double whole, rest;
    const E2m3Plan::Shape shape = cheapest(M, whole);
    // the token rows that fill whole rounds of 256 x 256 tiles, and the others in a launch of their own, if that wins by 3 %
    const long long tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
    const long long main_tile_rows = tiles_m * tiles_n / 256 * 256 / tiles_n;
    if (main_tile_rows > 0 && main_tile_rows < tiles_m) {
        const int rows_main = (int)main_tile_rows * 256;
        const E2m3Plan::Shape rest_shape = cheapest(M - rows_main, rest);
        const double divided = e2m3_shape_cost(E2m3Plan::k256, rows_main, N, K) + rest;
        if (divided < 0.97 * whole) {
            if (cost != nullptr) *cost = divided;
            return {E2m3Plan::k256, rows_main, rest_shape};
        }
    }
    if (cost != nullptr) *cost = whole;
    return {shape, M, shape};
}

// The kernel with the weights in registers (gemm_resident.h): 256 channels per block, the tokens in as many ranges of steps of 32 as fill the
// chip.  K where 64 channels of a wave fit beside two sets of results; affine codes are written for K = 1024 and 2048 only.  (K = 128 and 256 have few
// products per result: 40000 x 128 -> 2048 33.2 us in 256-row tiles, 31.8 in this one, 10992 x 256 -> 1024 8.1 / 8.9.)
constexpr bool e2m3_resident_k(int K, bool shifted)
{
    return K == 1024 || K == 2048 || (!shifted && (K == 512 || K == 768 || K == 1280 || K == 1536 || K == 1792));
}
// CT: a wave has 16 CT channels (a block four times that) and 128 / CT tokens a step
inline int resident_groups(int N, int CT = 4) { return (N + 64 * CT - 1) / (64 * CT); }
inline int resident_ranges(int M, int N, int CT = 4) { return std::max(1, std::min(256 / resident_groups(N, CT), (M + 128 / CT - 1) / (128 / CT))); }

// K = 1024, E2M3, no zero points: 128 channels a wave instead of 64 halve what a product reads from LDS and what comes from memory, and take 3 us more
// to load.  us, 64 / 128 channels: 4096 channels, 10992 tokens (22 steps of a block) 30.1 / 28.3, 24576 (48) 58.3 / 53.1, 65536 (128) 137 / 127; 3072, 16384 (25)
// 29.9 / 31.5, 24576 (37) 42.5 / 41.2, 65536 (98) 105 / 97; 2048, 32976 (33) 37.2 / 38.4, 65536 (64) 70.2 / 65.7; 1536, 65536 (49) 53.3 / 56.2; 1040, where the
// wider groups leave a third of the chip idle, 44.9 / 48.3; on another board 6144, 12288 50.6 / 46.7; 8192, 8192 44.1 / 41.9, 14000 70.4 / 65.8.  Beyond 8192
// channels it depends on how the groups divide the chip: 8208, 14000 74.9 / 67.4; 12288, 6000 47.0 / 48.2, 16000 115 / 108; 16384, 4608 47.9 / 51.3, 16000 147 / 140.
// At K = 768 and 512, which were built as well, equal or slower up to 65536 tokens.
inline bool resident_wide(int M, int N)
{
    auto steps = [&](int CT) { const int s = (M + 128 / CT - 1) / (128 / CT), r = resident_ranges(M, N, CT); return (s + r - 1) / r; };
    return N >= 2048 && N <= 8192 && steps(8) >= 36 && steps(8) <= steps(4);
}

// Its price in microseconds, to be compared with the tiles'.  Loading the weights into the registers costs 5.5 + 2.4 k before the first product, a
// step of a block 0.62 k, and writing Y 0.098 per megabyte on top of that.  Fitted to the products alone of 7 widths x 7 token counts at K = 512, 768 and 1024 (5 %, rms),
// with 1.5 us more before the first step as calls run it, behind kernel 1: without them calls of few steps lose (with kernel 1, 2355 x 1024 -> 704, two steps, 10.4 in
// tiles / 11.1 here, 585 x 1024 -> 2576 9.8 / 10.6).  Held against 1880 random calls of all seven K and of affine codes, with kernel 1 in front, that the two prices put within a
// third of each other: the choice is 0.5 % slower than the better of the two on geometric average; and 2 % faster than the choice among kernels on 32x32 instructions,
// 1 % of the calls being slower than by that one by 4 % and more (6441 x 768 -> 2336 21.6 / 23.2).
// us with kernel 1, tiles / this one: 6452 x 2048 -> 3552 46.7 / 42.2, 2872 x 1536 -> 2928 23.7 / 20.3, 3697 x 1280 -> 2576 26.7 / 21.7, 4791 x 1024 -> 2720 23.1 / 21.3,
// 7690 x 1024 -> 1920 23.4 / 21.1, 32648 x 1024 -> 448 39.9 / 35.4, 33436 x 1024 -> 256 34.1 / 34.6, 3617 x 2048 -> 3648 28.8 / 30.0.  us of the product, tiles / this one:
// 137400 x 1024 -> 4096 385 / 264, 32976 x 1024 -> 4096 90 / 71.6, 10992 x 1024 -> 4096 38.9 / 28, 10992 x 768 -> 3072 25.8 / 18.5, 4096 x 1024 -> 4096 15.9 / 13.5,
// 2048 x 1024 -> 4096 9.5 / 9.6.
inline double e2m3_resident_cost(int M, int N, int K)
{
    const double k = K / 1024.0;
    const int steps = (M + 31) / 32, ranges = resident_ranges(M, N);
    return 1.015 * (5.5 + 2.4 * k + 0.62 * k * ((steps + ranges - 1) / ranges) + 0.098e-6 * 2.0 * M * N);
}
// The tiles' price is too high where the rows of Y are 64-byte pieces but no whole lines (N = 32 mod 64), the more the shorter K.  Of 250 such calls within a sixth of each
// other, those that 1 + 61 / K puts on the wrong side cost 0.6 % in all; 1.12 for every K cost twice that (with kernel 1, tiles / this one: 48869 x 1024 -> 160 47.0 / 42.8,
// 23603 x 1024 -> 288 33.4 / 31.5; 4787 x 512 -> 3744 18.8 / 19.7).  K = 1280 alone is better off with it (37024 -> 224 63.8 / 65.9).
// This kernel's is too low where the weights are more than an XCD's L2 of 4 MiB holds with anything else, all of which read them all: 3617 x 2048 -> 3648 28.8 / 30.0,
// 3693 -> 3392 28.7 / 29.5, 3725 x 1792 -> 3200 31.4 / 32.1, of 380 calls of 1024 to 4096 channels in one round of tiles, the wrong side costs
// 0.4 % in all without the 1.04, 0.2 with it.
inline bool e2m3_resident(int M, int N, int K, bool shifted)
{
    if (!e2m3_resident_k(K, shifted)) return false;
    double tiles;
    e2m3_gemm_plan(M, N, K, &tiles);
    const double pieces = N % 64 != 32 ? 1.0 : K == 1280 ? 1.12 : 1.0 + 61.0 / K, spill = (long long)N * K > (4 << 20) ? 1.04 : 1.0;
    return e2m3_resident_cost(M, N, K) * pieces * spill < tiles;
}

// int8 blocks with the weights in registers: K = 1024, whose 256 channels take half of them (blocks come with K = 1024, 2048 and 4096; at 2048 they would
// take all).  Few tiles stay with the kernels made for them: alone, those take less than this one (2748 x 1024 7.7 / 9.0 us).  So do few tokens, whose
// time is the weights' (40 x 66064 20.6 / 22.1, 300 x 66064 49.6 / 43.9).  The others by price
// in microseconds.  The price is that of this kernel on the 32x32x32 instruction, fitted to 234 random problems of 100 to 137400 rows (its own within 5 %, rms), and a tenth
// to a fifth too high for the one that runs: calls priced level stay in tiles and are the slower for it (20000 x 512 16.1 / 13.7, 65536 x 1024 71.0 / 63.6).  256s cost 4 us more where the rows of Y are 32-byte
// pieces of lines, 1 where they are 64-byte ones (at 4 there too, one round of them with N = 32 mod 64 came here and lost: 2796 x 4576 23.6 / 27.5,
// 5567 x 2080 25.4 / 28.1, 10392 x 992 30.0 / 30.8).  As calls run it, behind kernel 1, the 1620 of 3000 other problems that it gives to this kernel are
// 1.18 times faster than in tiles on geometric average; 13 are slower by more than 2 %, by 6 % at worst (both kernels on 32x32x32).  us of the GEMM as they are now,
// tiles / this one: 137400 x 4096 561 / 452, 32976 x 4096 144 / 120, 32976 x 1024 43.4 / 33.2, 10992 x 3072 42.8 / 34.0.
inline bool i8b_resident(int M, int N, int K)
{
    if (K != 1024 || M < 256 || int8_instruction_few_tiles(M, N, K, 8, true) != FewTiles::kNone) return false;
    double tiles;
    const GemmPlan plan = int8_instruction_gemm_plan(M, N, K, 8, false, false, &tiles);
    if (plan.shape == GemmPlan::kDeep) return false;
    if (plan.shape == GemmPlan::kBig) tiles += N % 32 != 0 ? 4.0 : N % 64 != 0 ? 1.0 : 0.0;
    const int steps = (M + 31) / 32, ranges = resident_ranges(M, N);
    return 1.03 * (7.4 + 0.89 * ((steps + ranges - 1) / ranges) + 0.236e-6 * 2.0 * M * N) < tiles;
}

}  // namespace qvggt
