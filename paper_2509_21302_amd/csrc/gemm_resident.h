// Online kernel 2 with the weights resident in registers, for K that they have room for and enough tokens (e2m3_resident and i8b_resident in
// gemm_plan.h): E2M3 codes on the 6-bit floating-point matrix path, int8 codes on the int8 one.  Sums, results and operand formats are those of
// gemm_e2m3.hip and gemm_w4a4.hip, bit for bit.
//
// A wave keeps 64 channels of all K (E2M3: 12 registers a lane per 64 codes, 192 at K = 1024, 384 at 2048; int8: 256 at 1024) and the tokens go past it,
// 32 at a time: a step is K / 32 (int8 K / 16) MFMAs into 32 accumulator registers, and because that is all that a step's results take, there is a
// second set: the results of one step are scaled and stored between the MFMAs of the next.  That is what the 256 x 256 tiles cannot do, whose
// accumulators fill half the registers: the matrix pipes idle in their epilogue, two fifths of a tile at K = 1024 (int8: a third).  The tokens are also the only
// operand that moves (E2M3: 24 KiB per step of a block at K = 1024, where the tiles move 24 KiB per 64 codes of K), and a step is fine enough that
// the last round of a launch wastes little: the tokens are divided evenly, to 32.
//
// Four waves of 64 channels per block, one block per compute unit, one wave per SIMD.  Tokens go from memory straight into an LDS ring
// (global_load_lds_dwordx4); each wave reads a fragment for two MFMAs: 117 bytes of LDS traffic per cycle at the matrix rate, 144 in the tiles (int8: 80).
// The tokens are the MFMA's row operand, so that a lane holds one channel of each set and neighbouring channels of two sets are a dword of Y: no
// transposition, a store instruction writes two whole lines.
//
// What bounds it: the board's power.  137400 x 1024 -> 4096: 321 us (tiles 385), with all codes zero 233, without the stores 239, without stores and
// transfers 214, which is the register-only rate of the instruction (5.4 PFLOP/s); the stores alone take 181.  int8 codes: 527 us (tiles 637), codes
// of a sixteenth of the size 482 (548), all zero 328 (409); the register-only rate would be 340.  At 8 frames (10992 x 1024 -> 4096, 29 us, tiles
// 39) 6 us are the launch and the weights' way into the registers.  Tried and not better: pairs of dwords per store (two swaps more: 1 % slower),
// fragments read 4 to 7 units ahead instead of 3, stores of wider scope, a wait that counts the stores as well.
//
// The sizes are instantiated in several files, gemm_resident*.hip, which compile side by side (one file of all takes as long as the rest of the library).
#pragma once
#include "e2m3.h"
#include "gemm_plan.h"
#include "resident.h"

namespace qvggt {

typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v16i __attribute__((ext_vector_type(16)));

// 4 bytes per lane to base + lane_off, past the caches or through them
template <bool STREAM>
__device__ inline void store4(void *base, uint32_t lane_off, uint32_t v)
{
    if constexpr (STREAM) asm volatile("global_store_dword %0, %1, %2 nt" ::"v"(lane_off), "v"(v), "s"(base) : "memory");
    else asm volatile("global_store_dword %0, %1, %2" ::"v"(lane_off), "v"(v), "s"(base) : "memory");
}

// An operand format: a unit is what one MFMA takes of a row's codes, a K-tile of the format holds TILE_UNITS of them.
struct E2m3Codes {
    typedef v6i Weights;                                               // a lane's share of a unit
    typedef v8i Fragment;                                              // as the matrix builtin takes it: E2M3 numbers fill six of the eight registers
    typedef v16f Sums;
    static constexpr int TILE_UNITS = 1, ROW_BYTES = U_BYTES, WREGS = 6;
    static __device__ inline Sums multiply(Fragment f, Weights w, Sums s)
    {
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f, __builtin_shufflevector(w, w, 0, 1, 2, 3, 4, 5, -1, -1), s, 2, 2, 0, UNIT_SCALE_ONE, 0, UNIT_SCALE_ONE);
    }
    static __device__ inline uint32_t first(int r, int h) { return r * U_BYTES + h * 16; }        // a lane's 16 bytes of unit 0 (its other 8 are at 32 + 8 h of the row)
};
// "int8 blocks": K-tiles of 64 bytes a row, two units of 32 codes, four 16-byte chunks whose places are swizzled with bits 2 and 3 of the row
struct Int8Codes {
    typedef v4i Weights;
    typedef v4i Fragment;
    typedef v16i Sums;
    static constexpr int TILE_UNITS = 2, ROW_BYTES = 64, WREGS = 4;
    static __device__ inline Sums multiply(Fragment f, Weights w, Sums s) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(f, w, s, 0, 0, 0); }
    static __device__ inline uint32_t first(int r, int h) { return r * 64 + ((h ^ (r >> 2 & 3)) << 4); }      // unit 1: bit 5 the other way
};

// Pins values to one half of the register file at this point (accumulator and ordinary registers: the matrix instructions read either).
template <class V>
__device__ inline void keep_in_accumulators(V &a, V &b) { asm volatile("" : "+a"(a), "+a"(b)); }
template <class V>
__device__ inline void keep_in_registers(V &a, V &b) { asm volatile("" : "+v"(a), "+v"(b)); }
__device__ inline void keep_in_registers(float2 &a) { asm volatile("" : "+v"(a.x), "+v"(a.y)); }

// UNITS per ring stage, PARTS stages per step of 32 tokens: K = 64 * UNITS * PARTS (E2M3), 32 * UNITS * PARTS (int8)
template <class CODES, int UNITS, int PARTS>
struct ResidentCfg {
    static constexpr int NW = 4, THREADS = NW * 64;
    static constexpr int TILES = UNITS / CODES::TILE_UNITS, TILE_BYTES = 32 * CODES::ROW_BYTES;        // K-tiles of a stage, 32 rows of one
    static constexpr int RB_TILE = RB * CODES::ROW_BYTES;              // K-tile of a block of the operand format
    static constexpr int STAGE_BYTES = TILES * TILE_BYTES;
    static constexpr int STAGES = CODES::TILE_UNITS > 1 ? 8 : UNITS <= 16 ? 6 : 5;
    static constexpr int NT = STAGE_BYTES / 1024;                      // 1 KiB pieces of a stage
    static constexpr int LPW = (NT + NW - 1) / NW, LPW_MIN = NT / NW;  // pieces per wave
    static constexpr int SLOTS = 8, SLOT_BYTES = 512;                  // per step 32 token scales and (SHIFTED) 32 zero points, each twice
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + SLOTS * SLOT_BYTES;
    static_assert(UNITS % CODES::TILE_UNITS == 0 && STAGE_BYTES % 1024 == 0 && LDS_BYTES <= 160 * 1024, "whole K-tiles and pieces; one block per compute unit");
    // while stage q runs, the scales of stage q - 1 + STAGES arrive and those of the step before q's are read
    static_assert((STAGES - 2 + PARTS) / PARTS + 1 < SLOTS, "scales in use are not overwritten");
};

template <class CODES, int UNITS, int PARTS, bool SHIFTED, bool STREAM_Y>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void resident_gemm_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq, const float *__restrict__ sw,
    const uint16_t *__restrict__ bias, int M, int N, uint16_t *__restrict__ Y, const float *__restrict__ xzero, const float *__restrict__ wsum,
    int groups, int ranges)
{
    using C = ResidentCfg<CODES, UNITS, PARTS>;
    constexpr int ST = C::STAGES, LPW = C::LPW, ALL = UNITS * PARTS, TU = CODES::TILE_UNITS, ALL_TILES = ALL / TU;
    constexpr int WREGS = 2 * CODES::WREGS;                            // registers of a unit's weights
    constexpr bool TIGHT = ALL * WREGS > 336;                          // short of registers: scalar arithmetic for some addresses, scales at the last moment
    constexpr int R = UNITS % 4 == 0 ? 4 : 7, D = TIGHT && SHIFTED ? 2 : 3;                           // fragment buffers, units of look-ahead
    static_assert(UNITS % R == 0, "fragment buffers repeat with the stage");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;

    // XCD x (blocks are dealt round-robin to the 8 XCDs) has a contiguous range of tokens, all channel groups of which read it at one time
    const int id = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int range = id / groups, group = id - range * groups;
    if (range >= ranges) return;
    const int steps = (M + 31) >> 5;
    const int step0 = (int)((long long)range * steps / ranges), step1 = (int)((long long)(range + 1) * steps / ranges);
    if (step0 >= step1) return;

    // ---- tokens -> LDS.  A stage holds K-tiles of 32 rows (E2M3 1.5 KiB, int8 2 KiB), each contiguous in memory and in the stage
    constexpr int WHOLE = CODES::ROW_BYTES == 48 ? 3 : 1, WHOLE_TILES = WHOLE * C::NW * 1024 / C::TILE_BYTES;
    constexpr int NOFF = TIGHT || TU > 1 ? WHOLE : LPW;     // a wave's piece i + WHOLE is its piece i of WHOLE_TILES K-tiles later
    static_assert(WHOLE * C::NW * 1024 % C::TILE_BYTES == 0, "pieces repeat with whole K-tiles");
    uint32_t off[NOFF];
#pragma unroll
    for (int i = 0; i < NOFF; ++i) {
        const int q = (i * C::NW + wave) * 64 + lane;                  // 16-byte chunk of the stage
        off[i] = (uint32_t)(q / (C::TILE_BYTES / 16)) * C::RB_TILE + (uint32_t)(q % (C::TILE_BYTES / 16)) * 16;
    }
    int ld_step = step0, ld_part = 0, ld_slot = 0;
    const uint32_t dst0 = lds0 + wave * 1024;
    uint32_t ld_dst = dst0;                                            // this wave's first piece of the ring stage to fill
    const uint8_t *ld_base = Xq + (size_t)(step0 >> 2) * ALL_TILES * C::RB_TILE + (step0 & 3) * C::TILE_BYTES;
    auto issue_piece = [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        const uint8_t *base = ld_base + i / NOFF * WHOLE_TILES * C::RB_TILE;
        if constexpr ((i + 1) * C::NW <= C::NT) dma16_at<i * C::NW * 1024>(off[i % NOFF], base, ld_dst);
        else if (i * C::NW + wave < C::NT) dma16_at<i * C::NW * 1024>(off[i % NOFF], base, ld_dst);       // wave-uniform
    };
    auto issue_scales = [&]() {                                        // before the pieces of its stage: landed when they have
        if (ld_part == 0 && wave == C::NW - 1) {
            const uint32_t token = (uint32_t)min(ld_step * 32 + c, M - 1) * 4, dst = lds0 + ST * C::STAGE_BYTES + ld_slot * C::SLOT_BYTES;
            dma4(token, sx, dst);
            if constexpr (SHIFTED) dma4(token, xzero, dst + 256);
        }
    };
    auto advance = [&]() {
        ld_dst = ld_dst == dst0 + (ST - 1) * C::STAGE_BYTES ? dst0 : ld_dst + C::STAGE_BYTES;
        if (PARTS > 1 && ++ld_part < PARTS) { ld_base += C::TILES * C::RB_TILE; return; }
        ld_part = 0;
        ld_base -= (PARTS - 1) * C::TILES * C::RB_TILE;
        ld_slot = (ld_slot + 1) & (C::SLOTS - 1);
        if (ld_step < step1 - 1) {                                     // past the last step: it again (never used)
            ++ld_step;
            ld_base += (ld_step & 3) != 0 ? C::TILE_BYTES : ALL_TILES * C::RB_TILE - 3 * C::TILE_BYTES;
        }
    };
    auto issue_stage = [&]() {
        issue_scales();
        e_static_for<LPW>([&](auto i_c) { issue_piece(i_c); });
        advance();
    };

    // ---- weights.  A lane's two columns (MFMA column c of accumulators 0 and 1) are neighbouring channels of the wave's 64, so that its pair of
    // results is a dword of Y and 32 lanes store a line of it.  32 consecutive rows are loaded at a time, even ones to lanes 0 .. 15, odd ones
    // to lanes 16 .. 31, and a swap of rows of 16 lanes pairs them: rows 2 c and 2 c + 1 in one load instruction each are twice the lines (K = 1024:
    // all weights 2.8 us, and 1.9 + 0.4 this way).  Past the last channel the wave's others again: the same values to the same places
    const int ch0 = group * 256 + wave * 64;
    const bool idle = ch0 >= N;
    const int chans = min(N - ch0, 64);
    issue_stage();
    issue_stage();
    const int chan = idle ? 0 : ch0 + 2 * c % chans;
    float2 swv = *reinterpret_cast<const float2 *>(sw + chan);
    float2 bv = make_float2(0.0f, 0.0f), wsv = make_float2(0.0f, 0.0f);
    if (bias != nullptr) {
        const uint32_t b = *reinterpret_cast<const uint32_t *>(bias + chan);
        bv = make_float2(__uint_as_float(b << 16), __uint_as_float(b & 0xFFFF0000u));
    }
    if constexpr (SHIFTED) wsv = *reinterpret_cast<const float2 *>(wsum + chan);
    typename CODES::Weights W[2][ALL];
    if (!idle) {
        const uint8_t *p[2][TU];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = ch0 + (32 * j + 2 * (c & 15) + (c >> 4)) % chans;
#pragma unroll
            for (int t = 0; t < TU; ++t) p[j][t] = Wq + (size_t)(r / RB) * ALL_TILES * C::RB_TILE + (CODES::first(r % RB, h) ^ t << 5);
        }
        auto load = [&](auto u_c) {
            constexpr int u = decltype(u_c)::value;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const v4i lo = *reinterpret_cast<const v4i *>(p[j][u % TU] + u / TU * C::RB_TILE);
                if constexpr (CODES::WREGS == 6) {
                    const int2 hi = *reinterpret_cast<const int2 *>(p[j][0] + u * C::RB_TILE + 32 - h * 8);
                    W[j][u] = v6i{lo[0], lo[1], lo[2], lo[3], hi.x, hi.y};
                } else {
                    W[j][u] = lo;
                }
            }
        };
        constexpr int AHEAD = TU * (TIGHT ? 8 : ALL_TILES < 14 ? ALL_TILES : 14);     // 56 loads in flight; 32 where the registers do not hold more
        e_static_for<AHEAD>(load);
        e_static_for<ALL>([&](auto u_c) {
            constexpr int u = decltype(u_c)::value;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < CODES::WREGS; ++e) {
                const auto s = __builtin_amdgcn_permlane16_swap((uint32_t)W[0][u][e], (uint32_t)W[1][u][e], false, false);
                W[0][u][e] = (int)s[0];
                W[1][u][e] = (int)s[1];
            }
            // where they stay; without a word the compiler moves some of them about in the loop (60 moves a step, 5 % of the kernel)
            if constexpr ((u + 1) * WREGS <= 252) keep_in_accumulators(W[0][u], W[1][u]);
            else keep_in_registers(W[0][u], W[1][u]);
            if constexpr (u + AHEAD < ALL) load(std::integral_constant<int, u + AHEAD>{});
        });
    }
    // Stage q of the stream lives in ring stage q % ST.  Its fragments are read while it and the end of the stage before it are multiplied, so
    // behind the barrier that opens stage q the ring stage of q - 1 is free: it is refilled with stage q - 1 + ST
    e_wait_vmcnt<0>();                                                 // the first two stages, issued before the weights
    keep_in_registers(swv);                                            // here: the compiler would wait for them in the loop, and for all transfers with them
    keep_in_registers(bv);
    if constexpr (SHIFTED) keep_in_registers(wsv);
    __syncthreads();
#pragma unroll
    for (int s = 2; s < ST - 1; ++s) issue_stage();
    if (idle) {                                                        // no channels of its own: it moves its share of the tokens
        for (int s = (step1 - step0) * PARTS; s > 0; --s) {
            e_wait_vmcnt<(ST - 3) * C::LPW_MIN>();
            __syncthreads();
            issue_stage();
        }
        e_wait_vmcnt<0>();
        return;
    }

    // ---- fragments of the tokens
    typename CODES::Fragment F[R];
    if constexpr (TU == 1) {
#pragma unroll
        for (int f = 0; f < R; ++f) { F[f][6] = 0; F[f][7] = 0; }
    }
    const uint32_t frag = CODES::first(c, h), h8 = h * 8;
    auto read_lo = [&](auto f_c, int u, const uint8_t *stage) {
        constexpr int f = decltype(f_c)::value;
        const v4i v = *reinterpret_cast<const v4i *>(stage + (frag ^ u % TU << 5) + u / TU * C::TILE_BYTES);
        F[f][0] = v[0]; F[f][1] = v[1]; F[f][2] = v[2]; F[f][3] = v[3];
    };
    auto read_hi = [&](auto f_c, int u, const uint8_t *stage) {
        if constexpr (CODES::WREGS == 6) {
            constexpr int f = decltype(f_c)::value;
            const int2 v = *reinterpret_cast<const int2 *>(stage + frag + 32 - h8 + u * C::TILE_BYTES);
            F[f][4] = v.x; F[f][5] = v.y;
        }
    };

    // ---- results: register r of an accumulator is token 8 (r / 4) + 4 h + r % 4 of the step
    typename CODES::Sums acc[2][2];
    float4 st[4], zt[SHIFTED ? 4 : 1];
    int cs = 0, slot = 0;                                              // ring stage being multiplied (its LDS offset), scales of the step whose results leave
    const uint32_t row_bytes = (uint32_t)N * 2;
    uint8_t *yrow = reinterpret_cast<uint8_t *>(Y) + (size_t)step0 * 32 * row_bytes;      // of the next results to leave
    constexpr int NY = TIGHT ? 1 : 4;
    uint32_t y_off[NY];
#pragma unroll
    for (int r = 0; r < NY; ++r) y_off[r] = (uint32_t)chan * 2 + (uint32_t)(4 * h + r) * row_bytes;
    auto read_scales = [&](int q) {
        const uint8_t *p = smem + ST * C::STAGE_BYTES + slot * C::SLOT_BYTES + (8 * q + 4 * h) * 4;
        st[q] = *reinterpret_cast<const float4 *>(p);
        if constexpr (SHIFTED) zt[q] = *reinterpret_cast<const float4 *>(p + 256);
    };
    auto result = [&](auto b_c, int r) {
        constexpr int b = decltype(b_c)::value;
        const float s = (&st[r / 4].x)[r % 4];
        float a0 = (float)acc[b][0][r], a1 = (float)acc[b][1][r];
        if constexpr (SHIFTED) {
            const float z = 7.5f - (&zt[r / 4].x)[r % 4];
            a0 = fmaf(z, wsv.x, a0);
            a1 = fmaf(z, wsv.y, a1);
        }
        return pack_bf16x2(fmaf(a0, swv.x * s, bv.x), fmaf(a1, swv.y * s, bv.y));
    };

    // One stage: 2 UNITS slots of {one MFMA, a share of the side work}: the fragments D units ahead, the transfers of a later stage, and
    // the results of the step before (accumulators b ^ 1)
    auto stage = [&](auto b_c, auto part_c, auto first_c) {
        constexpr int b = decltype(b_c)::value, part = decltype(part_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;
        e_wait_vmcnt<(ST - 3) * C::LPW_MIN>();
        __syncthreads();
        const int ns = cs == (ST - 1) * C::STAGE_BYTES ? 0 : cs + C::STAGE_BYTES;
        const uint8_t *from = smem + cs;
        const typename CODES::Sums zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        if constexpr (!FIRST && part == 0) read_scales(0);
        e_static_for<2 * UNITS>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value, u = t / 2, j = t % 2, un = u + D;
            acc[b][j] = CODES::multiply(F[u % R], W[j][part * UNITS + u], part == 0 && u == 0 ? zero : acc[b][j]);
            using FB = std::integral_constant<int, un % R>;
            if constexpr (un == UNITS && j == 0) from = smem + ns;
            if constexpr (j == 0) read_lo(FB{}, un % UNITS, from);
            else read_hi(FB{}, un % UNITS, from);
            if constexpr (t == 0) issue_scales();
            e_static_for<LPW>([&](auto n_c) {
                constexpr int n = decltype(n_c)::value;
                if constexpr ((2 * n + 1) * 2 * UNITS / (2 * LPW) == t) issue_piece(n_c);
            });
            if constexpr (!FIRST) {
                e_static_for<16>([&](auto r_c) {
                    constexpr int r = decltype(r_c)::value, at = (2 * r + 1) * ALL / 16 - part * 2 * UNITS;     // spread over the step's 2 ALL slots
                    if constexpr (at == t) {
                        if constexpr (r % 4 == (TIGHT && SHIFTED ? 3 : 0) && r < 12) read_scales(r / 4 + 1);
                        store4<STREAM_Y>(yrow, y_off[r % NY], result(std::integral_constant<int, b ^ 1>{}, r));
                        if constexpr (r % 4 == 3) yrow += (TIGHT ? 5 : 8) * (size_t)row_bytes;
                        else if constexpr (TIGHT) yrow += row_bytes;
                    }
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        advance();
        cs = ns;
    };
    auto step = [&](auto b_c, auto first_c) {
        e_static_for<PARTS>([&](auto part_c) { stage(b_c, part_c, first_c); });
        if constexpr (!decltype(first_c)::value) slot = (slot + 1) & (C::SLOTS - 1);
    };
    auto last_results = [&](auto b_c) {
        const int left = M - (step1 - 1) * 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) read_scales(q);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t v = result(b_c, r);
            if (8 * (r / 4) + 4 * h + r % 4 < left) *reinterpret_cast<uint32_t *>(yrow + (8 * (r / 4) + r % 4) * (size_t)row_bytes + y_off[0]) = v;
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

template <class CODES, int UNITS, int PARTS, bool SHIFTED>
hipError_t launch_resident(const ResidentProblem &p, hipStream_t stream)
{
    using C = ResidentCfg<CODES, UNITS, PARTS>;
    const auto kern = e2m3_streams_y(p.M, p.N) ? resident_gemm_kernel<CODES, UNITS, PARTS, SHIFTED, true> : resident_gemm_kernel<CODES, UNITS, PARTS, SHIFTED, false>;
    const int groups = resident_groups(p.N), ranges = resident_ranges(p.M, p.N);
    kern<<<(groups * ranges + 7) / 8 * 8, C::THREADS, C::LDS_BYTES, stream>>>(p.Xq, p.sx, p.Wq, p.sw, p.bias, p.M, p.N, p.Y, p.xzero, p.wsum, groups, ranges);
    return hipGetLastError();
}
// the kernels of a size, for the list of those that need more dynamic LDS
#define QVGGT_RESIDENT(CODES, UNITS, PARTS, SHIFTED)                                                                                                       \
    {reinterpret_cast<const void *>(resident_gemm_kernel<CODES, UNITS, PARTS, SHIFTED, true>), ResidentCfg<CODES, UNITS, PARTS>::LDS_BYTES}, \
    {reinterpret_cast<const void *>(resident_gemm_kernel<CODES, UNITS, PARTS, SHIFTED, false>), ResidentCfg<CODES, UNITS, PARTS>::LDS_BYTES}

}  // namespace qvggt
