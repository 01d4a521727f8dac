// Online kernel 2 with the weights resident in registers, for K that they have room for and enough tokens (e2m3_resident and i8b_resident in
// gemm_plan.h): E2M3 codes on the 6-bit floating-point matrix path, int8 codes on the int8 one.  Sums, results and operand formats are those of
// gemm_e2m3.hip and gemm_w4a4.hip, bit for bit.
//
// A wave keeps 64 channels of all K (E2M3: 12 registers a lane per 64 codes, 192 at K = 1024, 384 at 2048; int8: 256 at 1024), or 128 of K = 1024 where
// that pays (resident_wide), and the tokens go past it, 32 or 16 at a time: a step is 64 MFMAs of K = 1024 into 32 accumulator registers, and because that is
// all that a step's results take, there is a second set: the results of one step are scaled and stored between the MFMAs of the next.  That is what the
// 256 x 256 tiles cannot do, whose accumulators fill half the registers: the matrix pipes idle in their epilogue, two fifths of a tile at K = 1024 (int8: a
// third).  The tokens are also the only operand that moves (E2M3: 24 KiB, or 12, per step of a block at K = 1024, where the tiles move 24 KiB per 64 codes of K),
// and a step is fine enough that the last round of a launch wastes little: the tokens are divided evenly.
//
// Four waves per block, one block per compute unit, one wave per SIMD.  Tokens go from memory straight into an LDS ring (global_load_lds_dwordx4).  They
// are the MFMA's row operand, and a lane's columns are neighbouring channels: no transposition, a store instruction writes four whole lines or eight.
//
// The MFMAs are the 16 x 16 ones: the board's power is what bounds this kernel, and they need less of it.  A register-only loop on codes of a normal
// distribution runs at 7.4 PFLOP/s with 16x16x128 and at 6.7 with 32x32x64 (int8 codes 4.1 and 3.5 POP/s).  fragments.h has where a
// lane reads.  What one wave per SIMD issues is the next limit: an MFMA of 16 cycles hides two other
// instructions that do not wait for each other, each further one costs 4 cycles, 8 if it needs the result of the one before.  So a result's
// instructions are dealt out over four slots, and the scalar bookkeeping over the stage.
//
// us, 137400 x 1024 -> 4096 on one box, 32x32 MFMAs 306, 64 channels a wave 290, 128 channels 264 (half the LDS reads and transfers per product; without
// stores 64 channels 224, also without the results' arithmetic 195, MFMAs alone 165; the stores alone take 181); 32976 tokens 79 / 75.5 / 71.6.  int8 codes: 24 frames
// of fc1 and fc2 with kernel 1 343 -> 333.  Tried and not better: fragments read 4 to 7 units ahead instead of 3, stores of wider scope, a wait that
// counts the stores as well.  K = 2048 reads its fragments two ahead: with three it needs 28 bytes of scratch memory a lane, affine codes 76.
//
// The sizes are instantiated in several files, gemm_resident*.hip, which compile side by side (one file of all takes as long as the rest of the library).
#pragma once
#include "e2m3.h"
#include "fragments.h"
#include "gemm_plan.h"
#include "resident.h"

namespace qvggt {

typedef int v6i __attribute__((ext_vector_type(6)));

// 8 or 16 bytes per lane to base + lane_off, past the caches or through them.  A store of more than 8 wants two wait states before its registers are
// written again (the compiler puts s_nop 1 behind its own), which the compiler does not put behind an asm block.
template <bool STREAM>
__device__ inline void store_row(void *base, uint32_t lane_off, const uint32_t (&v)[2])
{
    const uint64_t w = (uint64_t)v[1] << 32 | v[0];
    if constexpr (STREAM) asm volatile("global_store_dwordx2 %0, %1, %2 nt" ::"v"(lane_off), "v"(w), "s"(base) : "memory");
    else asm volatile("global_store_dwordx2 %0, %1, %2" ::"v"(lane_off), "v"(w), "s"(base) : "memory");
}
template <bool STREAM>
__device__ inline void store_row(void *base, uint32_t lane_off, const uint32_t (&v)[4])
{
    const v4i w = {(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
    if constexpr (STREAM) asm volatile("global_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1" ::"v"(lane_off), "v"(w), "s"(base) : "memory");
    else asm volatile("global_store_dwordx4 %0, %1, %2\n\ts_nop 1" ::"v"(lane_off), "v"(w), "s"(base) : "memory");
}

// An operand format.  A fragment is what an MFMA takes of 16 rows: 128 codes of each in E2M3 (two K-tiles of the format), 64 in int8 (one).  Lane l has
// row l % 16 and a quarter of its codes (fragments.h).  A step of 32 tokens has as many fragments as E2M3 K-tiles, twice as many as int8 ones (TILE_UNITS).
struct E2m3Codes {
    typedef v6i Weights;                                               // a lane's share of a fragment
    typedef v8i Fragment;                                              // as the matrix builtin takes it: E2M3 numbers fill six of the eight registers
    typedef v4f Sums;
    static constexpr int TILE_UNITS = 1, ROW_BYTES = U_BYTES, WREGS = 6, KTILES = 2;
    static __device__ inline Sums multiply(Fragment f, Weights w, Sums s)
    {
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f, __builtin_shufflevector(w, w, 0, 1, 2, 3, 4, 5, -1, -1), s, 2, 2, 0, UNIT_SCALE_ONE, 0, UNIT_SCALE_ONE);
    }
    static __device__ inline uint32_t place(int r, int q, int tile_bytes) { return e2m3_place(r, q, tile_bytes); }
};
// "int8 blocks": K-tiles of 64 bytes a row
struct Int8Codes {
    typedef v4i Weights;
    typedef v4i Fragment;
    typedef v4i Sums;
    static constexpr int TILE_UNITS = 2, ROW_BYTES = 64, WREGS = 4, KTILES = 1;
    static __device__ inline Sums multiply(Fragment f, Weights w, Sums s) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(f, w, s, 0, 0, 0); }
    static __device__ inline uint32_t place(int r, int q, int) { return i8_place(r, q); }
};

// Pins values to one half of the register file at this point (accumulator and ordinary registers: the matrix instructions read either).
template <class V>
__device__ inline void keep_in_accumulators(V &a) { asm volatile("" : "+a"(a)); }
// Values that are worked out here, not where they are used (an instruction that waits for the one before it costs the wave twice the time)
__device__ inline void stay(float &a, float &b) { asm volatile("" : "+v"(a), "+v"(b)); }
template <class V>
__device__ inline void keep_in_registers(V &a) { asm volatile("" : "+v"(a)); }

// A wave has 16 CT channels (64 or 128) and 128 / CT tokens a step (32 or 16).
// UNITS fragments per ring stage and 16 tokens of the step, twice that for 32, PARTS stages per step: K = 64 * UNITS * PARTS (E2M3), 32 * UNITS * PARTS (int8)
template <class CODES, int UNITS, int PARTS, int CT>
struct ResidentCfg {
    static constexpr int NW = 4, THREADS = NW * 64;
    static constexpr int TOKENS = 128 / CT, CHANNELS = 16 * CT;        // of a step, of a wave
    static constexpr int TILES = UNITS / CODES::TILE_UNITS, TILE_BYTES = TOKENS * CODES::ROW_BYTES;    // K-tiles of a stage, the step's rows of one
    static constexpr int ALL_TILES = TILES * PARTS, KSTEPS = ALL_TILES / CODES::KTILES;
    static constexpr int RB_TILE = RB * CODES::ROW_BYTES;              // K-tile of a block of the operand format
    static constexpr int STAGE_BYTES = TILES * TILE_BYTES;
    static constexpr int STAGES = CODES::KTILES == 1 ? 8 : (UNITS <= 16 ? 6 : 5) * CT / 4;
    static constexpr int NT = STAGE_BYTES / 1024;                      // 1 KiB pieces of a stage
    static constexpr int LPW = (NT + NW - 1) / NW, LPW_MIN = NT / NW;  // pieces per wave
    static constexpr int STRIDE = STAGE_BYTES + 512;                   // room for a step's token scales and (SHIFTED) zero points behind it, 256 bytes each
    static constexpr int LDS_BYTES = STAGES * STRIDE;
    static_assert(CT == 4 || CT == 8, "a line of Y, or two, per token");
    static_assert(UNITS % CODES::TILE_UNITS == 0 && TILES % CODES::KTILES == 0 && STAGE_BYTES % 1024 == 0 && LDS_BYTES <= 160 * 1024,
                  "whole K-steps and pieces; one block per compute unit");
    static_assert(PARTS == 1 || (PARTS == 2 && STAGES % 2 == 0), "a ring stage is always the same part of a step");
    // the weights' way in: a ring of W_SLOTS K-tiles per wave behind the first two stages
    static constexpr int W_TILE = CHANNELS * CODES::ROW_BYTES, W_PIECES = W_TILE / 1024;
    static constexpr int W_FIT = (STAGES - 2) * STRIDE / (NW * W_TILE) / CODES::KTILES * CODES::KTILES;
    static constexpr int W_SLOTS = W_FIT < ALL_TILES ? W_FIT : ALL_TILES;
    static_assert(W_SLOTS >= CODES::KTILES, "a K-step of weights has room");
};

template <class CODES, int UNITS, int PARTS, int CT, bool SHIFTED, bool STREAM_Y>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void resident_gemm_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq, const float *__restrict__ sw,
    const uint16_t *__restrict__ bias, int M, int N, uint16_t *__restrict__ Y, const float *__restrict__ xzero, const float *__restrict__ wsum,
    int groups, int ranges)
{
    using C = ResidentCfg<CODES, UNITS, PARTS, CT>;
    constexpr int ST = C::STAGES, LPW = C::LPW, TU = CODES::TILE_UNITS, ALL_TILES = C::ALL_TILES, KSTEPS = C::KSTEPS, TOKENS = C::TOKENS;
    constexpr int GROUPS = TOKENS / 16, FRAGS = C::TILES / CODES::KTILES * GROUPS;                    // fragments of a stage
    constexpr bool TIGHT = KSTEPS * CT * CODES::WREGS > 336;           // short of registers: scalar arithmetic for some addresses
    constexpr int R = CT == 8 ? 2 : FRAGS % 4 == 0 ? 4 : 7, D = CT == 8 ? 1 : TIGHT ? 2 : 3;             // fragment buffers, fragments of look-ahead
    static_assert(FRAGS % R == 0, "fragment buffers repeat with the stage");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;

    // XCD x (blocks are dealt round-robin to the 8 XCDs) has a contiguous range of tokens, all channel groups of which read it at one time
    const int id = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int range = id / groups, group = id - range * groups;
    if (range >= ranges) return;
    const int steps = (M + TOKENS - 1) / TOKENS;
    const int step0 = (int)((long long)range * steps / ranges), step1 = (int)((long long)(range + 1) * steps / ranges);
    if (step0 >= step1) return;

    // ---- tokens -> LDS.  A stage holds K-tiles of the step's rows, each contiguous in memory and in the stage
    constexpr int WHOLE = CODES::ROW_BYTES == 48 ? 3 : 1, WHOLE_TILES = WHOLE * C::NW * 1024 / C::TILE_BYTES;
    constexpr int NOFF = TIGHT || TU > 1 ? WHOLE : LPW;     // a wave's piece i + WHOLE is its piece i of WHOLE_TILES K-tiles later
    static_assert(WHOLE * C::NW * 1024 % C::TILE_BYTES == 0, "pieces repeat with whole K-tiles");
    uint32_t off[NOFF];
#pragma unroll
    for (int i = 0; i < NOFF; ++i) {
        const int q = (i * C::NW + wave) * 64 + lane;                  // 16-byte chunk of the stage
        off[i] = (uint32_t)(q / (C::TILE_BYTES / 16)) * C::RB_TILE + (uint32_t)(q % (C::TILE_BYTES / 16)) * 16;
    }
    const uint32_t dst0 = lds0 + wave * 1024;                          // this wave's first piece of ring stage 0
    constexpr int SPB = RB / TOKENS;                                   // steps of a block of rows
    int ld_step = step0;
    const uint8_t *ld_base = Xq + (size_t)(step0 / SPB) * ALL_TILES * C::RB_TILE + step0 % SPB * C::TILE_BYTES;
    auto issue_piece = [&](auto i_c, uint32_t dst) {
        constexpr int i = decltype(i_c)::value;
        const uint8_t *base = ld_base + i / NOFF * WHOLE_TILES * C::RB_TILE;
        if constexpr ((i + 1) * C::NW <= C::NT) dma16_at<i * C::NW * 1024>(off[i % NOFF], base, dst);
        else if (i * C::NW + wave < C::NT) dma16_at<i * C::NW * 1024>(off[i % NOFF], base, dst);       // wave-uniform
    };
    auto after = [&](int stage) { return stage == (ST - 1) * C::STRIDE ? 0 : stage + C::STRIDE; };
    // a step's scales: behind its one stage; steps of two stages take the places in turn, a place lasting until the middle of the next step
    int ld_sc = 0;
    auto issue_scales = [&](auto part_c, int stage) {                  // before the pieces of the step's first stage: landed when they have
        if constexpr (decltype(part_c)::value == 0) {
            if (wave == C::NW - 1) {
                const uint32_t token = (uint32_t)min(ld_step * TOKENS + lane % TOKENS, M - 1) * 4, dst = lds0 + (PARTS == 1 ? stage : ld_sc) + C::STAGE_BYTES;
                dma4(token, sx, dst);
                if constexpr (SHIFTED) dma4(token, xzero, dst + 256);
            }
            if constexpr (PARTS > 1) ld_sc = after(ld_sc);
        }
    };
    // to the next stage's tokens, in three pieces that the loop does apart from each other; past the last step: it again (never used)
    int ld_move = 0;
    auto advance = [&](auto part_c, int piece) {
        constexpr bool LAST = decltype(part_c)::value == PARTS - 1;
        if (piece == 0) {
            if constexpr (LAST) ld_move = (ld_step & (SPB - 1)) == SPB - 1 ? ALL_TILES * C::RB_TILE - (SPB - 1) * C::TILE_BYTES : C::TILE_BYTES;
            else ld_move = C::TILES * C::RB_TILE;
        } else if (piece == 1) {
            if constexpr (LAST) {
                const int next = min(ld_step + 1, step1 - 1);
                ld_move = (next == ld_step ? 0 : ld_move) - (PARTS - 1) * C::TILES * C::RB_TILE;
                ld_step = next;
            }
        } else {
            ld_base += ld_move;
        }
        asm volatile("" ::"s"(ld_move));
    };
    auto issue_stage = [&](auto part_c, int stage) __attribute__((always_inline)) {
        issue_scales(part_c, stage);
        e_static_for<LPW>([&](auto i_c) { issue_piece(i_c, dst0 + stage); });
        for (int piece = 0; piece < 3; ++piece) advance(part_c, piece);
    };

    // ---- weights.  A lane's CT columns (MFMA column c of accumulators 0 .. CT - 1) are neighbouring channels of the wave's, so that its results of a
    // token are 8 or 16 bytes of Y and 16 lanes store one line of it or two.  They come through LDS, where the stages behind the first two still
    // are free: contiguous KiBs in, each lane's rows CT c + j out.  Those rows lie 2 or 4 bank groups of 16 bytes apart modulo 16; to spread a read's 16 lanes over all
    // groups, the 16-byte chunks are turned within 64 or 128 bytes by an amount that goes up every 16 rows (E2M3), resp. rows swapped within four
    // (int8), which the transfer's lane offsets do for nothing.  (Loads of a lane's rows straight into the registers touch three times the lines: all
    // weights and the first tokens at K = 1024 7 us, this way 5.)  Past the last channel the wave's others again: the same values to the same places
    const int ch0 = group * (C::NW * C::CHANNELS) + wave * C::CHANNELS;
    const bool idle = ch0 >= N;
    const int chans = min(N - ch0, C::CHANNELS);
    issue_stage(std::integral_constant<int, 0>{}, 0);
    issue_stage(std::integral_constant<int, 1 % PARTS>{}, C::STRIDE);
    const int chan = idle ? 0 : ch0 + CT * c % chans;
    float swv[CT], bv[CT], wsv[SHIFTED ? CT : 1];
#pragma unroll
    for (int j = 0; j < CT; ++j) {
        swv[j] = sw[chan + j];
        bv[j] = bias != nullptr ? __uint_as_float((uint32_t)bias[chan + j] << 16) : 0.0f;
        if constexpr (SHIFTED) wsv[j] = wsum[chan + j];
    }
    typename CODES::Weights W[KSTEPS][CT];
    if (!idle) {
        const uint8_t *w_base = Wq + (size_t)(ch0 / RB) * ALL_TILES * C::RB_TILE + ch0 % RB * CODES::ROW_BYTES;
        const uint32_t w_lds = lds0 + 2 * C::STRIDE + wave * (C::W_SLOTS * C::W_TILE);
        uint32_t w_off[C::W_PIECES];
#pragma unroll
        for (int i = 0; i < C::W_PIECES; ++i) {
            const int at = i * 64 + lane;                              // chunk in LDS
            w_off[i] = 16 * (CODES::KTILES == 1 ? at ^ i << 2 : (at & ~(CT - 1)) | ((at - at / 48) & (CT - 1)));
        }
        auto issue_tile = [&](auto t_c) {
            constexpr int t = decltype(t_c)::value;
            e_static_for<C::W_PIECES>([&](auto i_c) {
                constexpr int i = decltype(i_c)::value;
                dma16_at<t % C::W_SLOTS * C::W_TILE + i * 1024>(w_off[i], w_base + t * C::RB_TILE, w_lds);
            });
        };
        e_static_for<C::W_SLOTS>(issue_tile);
        // where row r's chunk `part` of a K-tile is
        auto place = [&](int r, int part) {
            if constexpr (CODES::KTILES == 1) return (uint32_t)((r * 4 + part) ^ (r >> 4) << 2) * 16;
            else return (uint32_t)(((r * 3 + part) & ~(CT - 1)) | ((r * 3 + part + (r >> 4)) & (CT - 1))) * 16;
        };
        uint32_t from[CT], from_hi[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int r = CT * c % chans + j;
            if constexpr (CODES::KTILES == 1) {
                from[j] = place(r, i8_quarter(g) ^ (r >> 2 & 3));
            } else {
                from[j] = e2m3_tile(g) * C::W_TILE + place(r, e2m3_blob(g));
                from_hi[j] = e2m3_tile(g) * C::W_TILE + place(r, 2) + e2m3_blob(g) * 8;
            }
        }
        const uint8_t *const w_smem = smem + 2 * C::STRIDE + wave * (C::W_SLOTS * C::W_TILE);
        e_static_for<KSTEPS>([&](auto k_c) {
            constexpr int k = decltype(k_c)::value, next = (k + 1) * CODES::KTILES, issued = k * CODES::KTILES + C::W_SLOTS;
            e_wait_vmcnt<((issued < ALL_TILES ? issued : ALL_TILES) - next) * C::W_PIECES>();
            const uint8_t *const tile = w_smem + k * CODES::KTILES % C::W_SLOTS * C::W_TILE;
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                const v4i lo = *reinterpret_cast<const v4i *>(tile + from[j]);
                if constexpr (CODES::WREGS == 6) {
                    const int2 hi = *reinterpret_cast<const int2 *>(tile + from_hi[j]);
                    W[k][j] = v6i{lo[0], lo[1], lo[2], lo[3], hi.x, hi.y};
                } else {
                    W[k][j] = lo;
                }
            }
            // where they stay; without a word the compiler moves some of them about in the loop (60 moves a step, 5 % of the kernel).  Once they are there
            // the slots are free
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                if ((k * CT + j + 1) * CODES::WREGS <= 252) keep_in_accumulators(W[k][j]);
                else keep_in_registers(W[k][j]);
            }
            e_static_for<CODES::KTILES>([&](auto t_c) {
                constexpr int t = issued + decltype(t_c)::value;
                if constexpr (t < ALL_TILES) issue_tile(std::integral_constant<int, t>{});
            });
        });
    }
    // Stage q of the stream lives in ring stage q % ST.  Its fragments are read while it and the end of the stage before it are multiplied, so
    // behind the barrier that opens stage q the ring stage of q - 1 is free: it is refilled with stage q - 1 + ST
    e_wait_vmcnt<0>();                                                 // the first two stages, issued before the weights
#pragma unroll
    for (int j = 0; j < CT; ++j) {                                     // here: the compiler would wait for them in the loop, and for all transfers with them
        keep_in_registers(swv[j]);
        keep_in_registers(bv[j]);
        if constexpr (SHIFTED) keep_in_registers(wsv[j]);
    }
    __syncthreads();
    e_static_for<ST - 3>([&](auto s_c) {
        constexpr int q = decltype(s_c)::value + 2;
        issue_stage(std::integral_constant<int, q % PARTS>{}, q * C::STRIDE);
    });
    if (idle) {                                                        // no channels of its own: it moves its share of the tokens
        int ps = (ST - 1) * C::STRIDE;
        for (int s = step1 - step0; s > 0; --s)
            e_static_for<PARTS>([&](auto part_c) {
                e_wait_vmcnt<(ST - 3) * C::LPW_MIN>();
                asm volatile("s_barrier" ::: "memory");
                issue_stage(std::integral_constant<int, (decltype(part_c)::value + ST - 1) % PARTS>{}, ps);
                ps = after(ps);
            });
        e_wait_vmcnt<0>();
        return;
    }

    // ---- fragments of the tokens
    typename CODES::Fragment F[R];
    if constexpr (TU == 1) {
#pragma unroll
        for (int f = 0; f < R; ++f) { F[f][6] = 0; F[f][7] = 0; }
    }
    const uint32_t frag = CODES::place(c, g, C::TILE_BYTES), g8 = e2m3_blob(g) * 8;
    // fragment u of a stage: tokens 16 (u % GROUPS) .. of its K-step u / GROUPS
    constexpr auto place = [](int u) constexpr { return u / GROUPS * CODES::KTILES * C::TILE_BYTES + u % GROUPS * 16 * CODES::ROW_BYTES; };
    auto read_lo = [&](auto f_c, int u, const uint8_t *stage) {
        constexpr int f = decltype(f_c)::value;
        const v4i v = *reinterpret_cast<const v4i *>(stage + frag + place(u));
        F[f][0] = v[0]; F[f][1] = v[1]; F[f][2] = v[2]; F[f][3] = v[3];
    };
    auto read_hi = [&](auto f_c, int u, const uint8_t *stage) {
        if constexpr (CODES::WREGS == 6) {
            constexpr int f = decltype(f_c)::value;
            const int2 v = *reinterpret_cast<const int2 *>(stage + frag + 32 - g8 + place(u));
            F[f][4] = v.x; F[f][5] = v.y;
        }
    };

    // ---- results: register r of accumulator [i][j] is token 16 i + 4 g + r of the step, channel j of the lane's
    typename CODES::Sums acc[2][GROUPS][CT];
    // scales (and zero points) of the tokens whose results leave: read while the step before is multiplied into the other of two sets; where registers are short
    // and the places last (PARTS = 2), four tokens' at the last moment
    constexpr bool LATE = TIGHT && PARTS == 2;
    constexpr int NS = LATE ? 1 : GROUPS, NB = LATE ? 1 : 2;
    float4 st[NB][NS], zt[NB][NS];
    float m0, m1, y0, y1;
    uint32_t out[CT / 2];
    int ps = (ST - 1) * C::STRIDE, cs = 0, ns = 0;                     // ring stages: the one before, the one being multiplied, the next one
    int sc = ps;                                                       // scales of the step whose results leave
    const uint32_t row_bytes = (uint32_t)N * 2;
    uint8_t *yrow = reinterpret_cast<uint8_t *>(Y) + (size_t)step0 * TOKENS * row_bytes;      // of the next results to leave
    constexpr int NY = TIGHT ? 1 : 4;
    uint32_t y_off[NY];
#pragma unroll
    for (int r = 0; r < NY; ++r) y_off[r] = (uint32_t)chan * 2 + (uint32_t)(4 * g + r) * row_bytes;
    auto read_scales = [&](auto b_c, int i) {
        constexpr int b = decltype(b_c)::value % NB;
        const uint8_t *p = smem + sc + C::STAGE_BYTES + (16 * i + 4 * g) * 4;
        st[b][i % NS] = *reinterpret_cast<const float4 *>(p);
        if constexpr (SHIFTED) zt[b][i % NS] = *reinterpret_cast<const float4 *>(p + 256);
    };
    // channel j of token 16 (tok / 4) + 4 g + tok % 4
    auto scale = [&](auto b_c, int tok, int j) { return swv[j] * (&st[decltype(b_c)::value % NB][tok / 4 % NS].x)[tok % 4]; };
    auto result = [&](auto b_c, int tok, int j, float m) {
        constexpr int b = decltype(b_c)::value;
        float a = (float)acc[b][tok / 4][j][tok % 4];
        if constexpr (SHIFTED) a = fmaf(7.5f - (&zt[b % NB][tok / 4 % NS].x)[tok % 4], wsv[j], a);
        return fmaf(a, m, bv[j]);
    };

    // One stage: CT FRAGS slots of {one MFMA, a share of the side work}: the fragments D ahead, the transfers of a later stage, and
    // the results of the step before (accumulators b ^ 1)
    auto stage = [&](auto b_c, auto part_c, auto first_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value, part = decltype(part_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;
        e_wait_vmcnt<(ST - 3) * C::LPW_MIN>();
        constexpr int SLOTS = CT * FRAGS, ALL_SLOTS = SLOTS * PARTS, PERIOD = ALL_SLOTS / 16;
        constexpr int SCALES_BEFORE = LATE ? 1 : 8;                      // slots from the scales' reads to the end of the stage
        constexpr int READS_AFTER = SCALES_BEFORE / CT * (CODES::WREGS == 6 ? 2 : 1);      // the fragments' in these slots
        static_assert(PARTS == 2 || (SCALES_BEFORE % CT == 0 && READS_AFTER >= 2), "what the barrier may leave in flight is newer than the scales");
        // A barrier, and of the LDS reads in flight, all of which __syncthreads() waits for, only the older: the scales', whose place (PARTS = 1) is
        // written during this stage.  The READS_AFTER behind them are fragments of the stage just opened, which nothing overwrites before the next barrier; half of them
        // are waited for too, should the compiler have joined two.
        if constexpr (PARTS == 1) asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(READS_AFTER / 2) : "memory");
        asm volatile("s_barrier" ::: "memory");
        using LP = std::integral_constant<int, (part + ST - 1) % PARTS>;  // the part that ring stage ps is refilled with
        const uint8_t *from = smem + cs;
        const typename CODES::Sums zero = {0, 0, 0, 0};
        e_static_for<SLOTS>([&](auto t_c) __attribute__((always_inline)) {
            constexpr int t = decltype(t_c)::value, u = t / CT, i = u % GROUPS, j = t % CT, un = u + D;
            acc[b][i][j] = CODES::multiply(F[u % R], W[(part * FRAGS + u) / GROUPS][j], part == 0 && u < GROUPS ? zero : acc[b][i][j]);
            using FB = std::integral_constant<int, un % R>;
            if constexpr (un == FRAGS && j == 0) from = smem + ns;
            if constexpr (j == 2) read_lo(FB{}, un % FRAGS, from);
            else if constexpr (j == 3) read_hi(FB{}, un % FRAGS, from);
            if constexpr (t == 2) issue_scales(LP{}, ps);
            if constexpr (t == 6) {
                ns = after(cs);
                asm volatile("" ::"s"(ns));
            }
            if constexpr (t == SLOTS - 13) advance(LP{}, 0);
            if constexpr (t == SLOTS - 9) advance(LP{}, 1);
            if constexpr (t == SLOTS - 5) advance(LP{}, 2);
            e_static_for<LPW>([&](auto n_c) {
                constexpr int n = decltype(n_c)::value;
                if constexpr (n * (SLOTS - 16) / LPW + 3 == t) issue_piece(n_c, dst0 + ps);
            });
            if constexpr (!FIRST) {
                e_static_for<16>([&](auto h_c) {                       // pairs of a lane's channels, each in four pieces
                    constexpr int hf = decltype(h_c)::value, tok = hf / (CT / 2), jp = hf % (CT / 2), at = hf * ALL_SLOTS / 16 - part * SLOTS;
                    using B = std::integral_constant<int, b ^ 1>;
                    if constexpr (at == t) {
                        m0 = scale(B{}, tok, 2 * jp);
                        m1 = scale(B{}, tok, 2 * jp + 1);
                        stay(m0, m1);
                    }
                    if constexpr (at + 1 == t) {
                        y0 = result(B{}, tok, 2 * jp, m0);
                        y1 = result(B{}, tok, 2 * jp + 1, m1);
                        stay(y0, y1);
                    }
                    if constexpr (at + (PERIOD > 2 ? 2 : 1) == t) out[jp] = pack_bf16x2(y0, y1);
                    if constexpr (at + (PERIOD > 3 ? 3 : PERIOD - 1) == t && jp == CT / 2 - 1) {
                        store_row<STREAM_Y>(yrow, y_off[tok % NY], out);
                        if constexpr (tok % 4 == 3) yrow += (TIGHT ? 13 : 16) * (size_t)row_bytes;
                        else if constexpr (TIGHT) yrow += row_bytes;
                        if constexpr (tok == 3 && NS < GROUPS) read_scales(B{}, 1);
                    }
                });
            }
            if constexpr (t == SLOTS - SCALES_BEFORE && part == PARTS - 1) {      // for this step's results
                sc = PARTS == 1 ? cs : after(sc);
#pragma unroll
                for (int i = 0; i < NS; ++i) read_scales(b_c, i);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        ps = cs;
        cs = ns;
    };
    auto step = [&](auto b_c, auto first_c) __attribute__((always_inline)) {
        e_static_for<PARTS>([&](auto part_c) __attribute__((always_inline)) { stage(b_c, part_c, first_c); });
    };
    auto last_results = [&](auto b_c) __attribute__((always_inline)) {
        const int left = M - (step1 - 1) * TOKENS;
#pragma unroll
        for (int tok = 0; tok < 4 * GROUPS; ++tok) {
            if (tok % 4 == 0) read_scales(b_c, tok / 4);
            v4i v;
#pragma unroll
            for (int j = 0; j < CT; j += 2) v[j / 2] = (int)pack_bf16x2(result(b_c, tok, j, scale(b_c, tok, j)), result(b_c, tok, j + 1, scale(b_c, tok, j + 1)));
            const int row = 16 * (tok / 4) + tok % 4;
            if (row + 4 * g < left) {
                if constexpr (CT == 8) *reinterpret_cast<v4i *>(yrow + row * (size_t)row_bytes + y_off[0]) = v;
                else *reinterpret_cast<int2 *>(yrow + row * (size_t)row_bytes + y_off[0]) = make_int2(v[0], v[1]);
            }
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    e_static_for<D>([&](auto u_c) {
        read_lo(u_c, decltype(u_c)::value, smem);
        read_hi(u_c, decltype(u_c)::value, smem);
    });
    step(I0{}, std::true_type{});
    int left = step1 - step0 - 1;
    for (; left >= 2; left -= 2) {
        step(I1{}, std::false_type{});
        step(I0{}, std::false_type{});
    }
    if (left == 1) {
        step(I1{}, std::false_type{});
        last_results(I1{});
    } else {
        last_results(I0{});
    }
    e_wait_vmcnt<0>();      // transfers issued past the last step must not outlive the block's LDS allocation
}

template <class CODES, int UNITS, int PARTS, int CT, bool SHIFTED>
hipError_t launch_resident_tiles(const ResidentProblem &p, hipStream_t stream)
{
    using C = ResidentCfg<CODES, UNITS, PARTS, CT>;
    auto kern = resident_gemm_kernel<CODES, UNITS, PARTS, CT, SHIFTED, true>;
    if constexpr (CT == 4) {                                           // 128 channels a wave: for more bytes of Y than are left in the caches
        if (!e2m3_streams_y(p.M, p.N)) kern = resident_gemm_kernel<CODES, UNITS, PARTS, CT, SHIFTED, false>;
    }
    const int groups = resident_groups(p.N, CT), ranges = resident_ranges(p.M, p.N, CT);
    kern<<<(groups * ranges + 7) / 8 * 8, C::THREADS, C::LDS_BYTES, stream>>>(p.Xq, p.sx, p.Wq, p.sw, p.bias, p.M, p.N, p.Y, p.xzero, p.wsum, groups, ranges);
    return hipGetLastError();
}
template <class CODES, int UNITS, int PARTS, bool SHIFTED>
hipError_t launch_resident(const ResidentProblem &p, hipStream_t stream)
{
    return launch_resident_tiles<CODES, UNITS, PARTS, 4, SHIFTED>(p, stream);
}
// the kernels of a size, for the list of those that need more dynamic LDS
#define QVGGT_RESIDENT_TILES(CODES, UNITS, PARTS, CT, SHIFTED, STREAM_Y) \
    {reinterpret_cast<const void *>(resident_gemm_kernel<CODES, UNITS, PARTS, CT, SHIFTED, STREAM_Y>), ResidentCfg<CODES, UNITS, PARTS, CT>::LDS_BYTES}
#define QVGGT_RESIDENT(CODES, UNITS, PARTS, SHIFTED) QVGGT_RESIDENT_TILES(CODES, UNITS, PARTS, 4, SHIFTED, true), QVGGT_RESIDENT_TILES(CODES, UNITS, PARTS, 4, SHIFTED, false)

}  // namespace qvggt
