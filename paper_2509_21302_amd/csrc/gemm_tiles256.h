// Products in tiles of 256 tokens x 256 channels, E2M3 and int8 codes, K of 768 and more (e2m3_tiles256, i8b_tiles256): gemm_e2m3_256.hip and gemm_w4a4.hip have the kernels.
//
// Four waves per block and compute unit, each with 128 x 128 of the tile: 256 accumulator registers, the least operand traffic per MFMA that the register
// file allows.  Persistent blocks, XCD-contiguous tile ranges, operands from global memory straight into an LDS ring (global_load_lds_dwordx4, 1 KiB
// contiguous per wave instruction, here also contiguous in memory).  A ring stage is the memory image of the tile's rows of one K-step: token rows, then channel
// rows.  K-step p is in registers, p + 1 has landed and is read while p is multiplied, later ones are on their way, and p's stage is refilled.
//
// The MFMAs are the 16 x 16 ones.  On codes of a normal distribution the register-only rate under the board's power limit is 7.4 PFLOP/s with 16x16x128 (E2M3)
// and 6.7 with 32x32x64, 4.1 and 3.5 POP/s with 16x16x64 and 32x32x32 (int8).
// Epilogue: accumulators from AGPRs, scale + bias, bf16, 16 tokens x 64 channels at a time through a wave-private LDS tile, whose way back
// is hidden under the arithmetic of the next 16, stores of whole 128-byte lines.
#pragma once
#include "e2m3.h"
#include "fragments.h"
#include "gemm_plan.h"

namespace qvggt {

// An operand format: blocks of RB rows with the K-tiles outermost, ROW_BYTES of a row per K-tile.  A K-step is what an MFMA takes: KTILES K-tiles.  Lane (c, q) of a
// fragment has a quarter of row c's: 16 bytes at place() of the stage, and in E2M3 8 more.
struct E2m3Tiles {
    typedef v8i Fragment;
    typedef v4f Sums;
    typedef float Sum;
    static constexpr int ROW_BYTES = U_BYTES, KTILES = 2, STAGES = 3, REGS = 6;
    static __device__ inline Sums multiply(Fragment a, Fragment b, Sums s) { return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, s, 2, 2, 0, UNIT_SCALE_ONE, 0, UNIT_SCALE_ONE); }
    static __device__ inline int place(int c, int q, int tile_bytes) { return e2m3_place(c, q, tile_bytes); }
    static __device__ inline float sum(float a) { return a; }
};
// "int8 blocks"
struct Int8Tiles {
    typedef v4i Fragment;
    typedef v4i Sums;
    typedef int Sum;
    static constexpr int ROW_BYTES = 64, KTILES = 1, STAGES = 4, REGS = 4;
    static __device__ inline Sums multiply(Fragment a, Fragment b, Sums s) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, s, 0, 0, 0); }
    static __device__ inline int place(int c, int q, int) { return i8_place(c, q); }
    static __device__ inline float sum(int a) { return (float)a; }
};

// SHIFTED: affine codes, as in gemm_e2m3.hip
template <class CODES, bool SHIFTED>
struct Cfg256 {
    static constexpr int NW = 4, THREADS = NW * 64, TM = 8, TN = 8;    // sub-tiles of 16 x 16 per wave, 2 x 2 waves
    static constexpr int BM = 2 * TM * 16, BN = 2 * TN * 16, ROWS = BM + BN;
    static constexpr int KTILES = CODES::KTILES, RB_TILE = RB * CODES::ROW_BYTES;      // K-tiles of a K-step, K-tile of a block of the format
    static constexpr int TILE_BYTES = ROWS * CODES::ROW_BYTES, STAGE_BYTES = KTILES * TILE_BYTES, STAGES = CODES::STAGES;
    static constexpr int RB_PIECES = RB_TILE / 1024;
    static constexpr int XT = BM / RB * RB_PIECES, NT = ROWS / RB * RB_PIECES;         // 1 KiB pieces of a K-tile: the first XT are token rows
    static constexpr int LPW = NT / NW;                                // transfers per wave
    static constexpr int NM = TM * TN, NF = TM + TN;
    static constexpr int SC_SYM_BYTES = BM * 4 + BN * 4 + BN * 2;      // per tile: sx f32, sw f32, bias bf16 (as in memory)
    static constexpr int SC_SYM_GROUPS = BM / 64 + BN / 64 + BN / 128;
    static constexpr int SC_BYTES = SC_SYM_BYTES + (SHIFTED ? BM * 4 + BN * 4 : 0);     // then zero points f32, code sums f32
    static constexpr int SC_GROUPS = SC_SYM_GROUPS + (SHIFTED ? BM / 64 + BN / 64 : 0);
    // scales of the tile and of the next, or where LDS does not hold both of the tile alone.  They go out before the transfers of the tile's first K-step and have landed
    // when all but the transfers of STAGES - 2 steps have: at the opening of its step STAGES - 2
    static constexpr int SC_BUFFERS = SHIFTED ? 1 : 2;
    static_assert(TILES256_LEAST_K / 64 / KTILES >= STAGES - 1, "a tile of the least K has that step");
    static constexpr int EP_PITCH = 128 + 16, EP_BYTES = NW * 16 * EP_PITCH;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + SC_BUFFERS * SC_BYTES + EP_BYTES;
    static_assert(BM % RB == 0 && BN % RB == 0 && NT % NW == 0, "tiles are whole blocks of the operand format, and every wave has as many pieces");
    static_assert(LDS_BYTES <= 160 * 1024, "one block per compute unit");
};

// STREAM_Y: Y goes past the caches (e2m3_streams_y); a template argument, because the kernel that asks at run time is 8 % slower at 137400 x 1024 -> 4096
template <class CODES, bool DEBUG, bool SHIFTED, bool STREAM_Y>
__device__ __forceinline__ void tiles256(
    const uint8_t *__restrict__ Xf, const float *__restrict__ sx, const uint8_t *__restrict__ Wf,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int N, int K,
    uint16_t *__restrict__ Y, int32_t *__restrict__ acc_debug, int tiles_m, int tiles_n,
    const float *__restrict__ xzero, const float *__restrict__ wsum)
{
    using C = Cfg256<CODES, SHIFTED>;
    constexpr int TM = C::TM, TN = C::TN, NM = C::NM, NF = C::NF, LPW = C::LPW, MOVES = C::KTILES * LPW;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t *sc_all = smem + C::STAGES * C::STAGE_BYTES;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int ktiles = K >> 6, ksteps = ktiles / C::KTILES;
    const int ntiles = tiles_m * tiles_n;

    // tile assignment: XCD x (blocks are dealt round-robin to the 8 XCDs) owns a contiguous tile range, channels fastest
    const int per_xcd = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
    const int tile_end = min((xcd + 1) * per_xcd, ntiles);
    const int first_tile = xcd * per_xcd + slot;
    if (first_tile >= tile_end) return;
    const int last_tile = tile_end - 1 - ((tile_end - 1 - first_tile) % slots);

    // ---- global -> LDS transfers.  Piece n of a K-tile (1 KiB: 16-byte chunks 64 n .. 64 n + 63) is moved by wave n % 4 in its slot n / 4.  Pieces below XT are
    // token rows, the rest channel rows; the K-tiles of a 128-row block of the operand format lie RB_TILE apart.
    const int xblocks = (M + RB - 1) / RB, wblocks = (N + RB - 1) / RB;
    const uint8_t *src[LPW];                                    // wave-uniform: K-tile 0 of this wave's pieces of the tile under the load cursor
    uint32_t ld_off[C::KTILES];                                 // from there to the K-step's K-tiles
    int ld_tile = first_tile, ld_kstep = 0;
    const uint32_t dst0 = lds0 + wave * 1024;
    auto set_tile_pointers = [&](int t) {
        const int tm = t / tiles_n, tn = t % tiles_n;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int n = i * C::NW + wave;
            const bool is_x = n < C::XT;
            const int m = is_x ? n : n - C::XT;
            const int blk = (is_x ? tm * (C::BM / RB) : tn * (C::BN / RB)) + m / C::RB_PIECES, piece = m % C::RB_PIECES;      // past the operand's end: the last block again, results unused
            src[i] = (is_x ? Xf : Wf) + (size_t)min(blk, (is_x ? xblocks : wblocks) - 1) * ktiles * C::RB_TILE + piece * 1024;
        }
#pragma unroll
        for (int h = 0; h < C::KTILES; ++h) ld_off[h] = (uint32_t)lane * 16 + h * C::RB_TILE;
    };
    // transfer n of a K-step's
    auto issue_transfer = [&](auto n_c, uint32_t stage) __attribute__((always_inline)) {
        constexpr int n = decltype(n_c)::value, h = n / LPW, i = n % LPW;
        dma16_at<h * C::TILE_BYTES + i * C::NW * 1024>(ld_off[h], src[i], dst0 + stage);
    };
    auto advance_cursor = [&]() {
#pragma unroll
        for (int h = 0; h < C::KTILES; ++h) ld_off[h] += C::KTILES * C::RB_TILE;
        if (++ld_kstep == ksteps) {
            ld_kstep = 0;
            ld_tile = min(ld_tile + slots, last_tile);          // past the last tile: re-read it (never used), keeps the stream uniform
            set_tile_pointers(ld_tile);
        }
    };
    auto issue_scales = [&](int t, int sb) {
        const int tm = t / tiles_n, tn = t % tiles_n;
        const uint32_t dst = lds0 + C::STAGES * C::STAGE_BYTES + sb * C::SC_BYTES;
#pragma unroll
        for (int g = 0; g < C::SC_GROUPS; ++g) {
            if (g % C::NW != wave) continue;
            if (g < C::BM / 64) {
                dma4(sx + min(tm * C::BM + g * 64 + lane, M - 1), dst + g * 256);
            } else if (g < C::BM / 64 + C::BN / 64) {
                const int h = g - C::BM / 64;
                dma4(sw + min(tn * C::BN + h * 64 + lane, N - 1), dst + C::BM * 4 + h * 256);
            } else if (g < C::SC_SYM_GROUPS) {
                if (bias != nullptr) {
                    const int h = g - C::BM / 64 - C::BN / 64;      // 64 dwords = 128 bf16 values
                    dma4(reinterpret_cast<const uint32_t *>(bias) + min(tn * (C::BN / 2) + h * 64 + lane, N / 2 - 1), dst + C::BM * 4 + C::BN * 4 + h * 256);
                }
            } else if (g < C::SC_SYM_GROUPS + C::BM / 64) {
                const int h = g - C::SC_SYM_GROUPS;
                dma4(xzero + min(tm * C::BM + h * 64 + lane, M - 1), dst + C::SC_SYM_BYTES + h * 256);
            } else {
                const int h = g - C::SC_SYM_GROUPS - C::BM / 64;
                dma4(wsum + min(tn * C::BN + h * 64 + lane, N - 1), dst + C::SC_SYM_BYTES + C::BM * 4 + h * 256);
            }
        }
    };

    // ---- fragments: [buffer][W sub-tiles, then X sub-tiles]
    typename CODES::Sums acc[TN][TM];
    typename CODES::Fragment F[2][NF];
    if constexpr (CODES::REGS == 6) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int f = 0; f < NF; ++f) { F[b][f][6] = 0; F[b][f][7] = 0; }
    }
    const int c = lane & 15, q = lane >> 4;
    const int at = CODES::place(c, q, C::TILE_BYTES);
    const int w_lane = at + (C::BM + wn * TN * 16) * CODES::ROW_BYTES, x_lane = at + wm * TM * 16 * CODES::ROW_BYTES;
    const int hi = e2m3_rest(q);                                // from the lane's first 16 bytes to its last 8
    auto place = [](int f, const uint8_t *wp, const uint8_t *xp) __attribute__((always_inline)) { return (f < TN ? wp + f * 16 * CODES::ROW_BYTES : xp + (f - TN) * 16 * CODES::ROW_BYTES); };
    auto read_lo = [&](auto b_c, int f, const uint8_t *wp, const uint8_t *xp) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value;
        const v4i v = *reinterpret_cast<const v4i *>(place(f, wp, xp));
        F[b][f][0] = v[0]; F[b][f][1] = v[1]; F[b][f][2] = v[2]; F[b][f][3] = v[3];
    };
    auto read_hi = [&](auto b_c, int f, const uint8_t *wp, const uint8_t *xp) __attribute__((always_inline)) {
        if constexpr (CODES::REGS == 6) {
            constexpr int b = decltype(b_c)::value;
            const int2 v = *reinterpret_cast<const int2 *>(place(f, wp, xp) + hi);
            F[b][f][4] = v.x; F[b][f][5] = v.y;
        }
    };
    // One K-step: NM slots of {one MFMA, a share of the side work}: the transfers of K-step p + STAGES first, for they take longest, and the LDS reads of the
    // next K-step's fragments into the other buffer, in the order the MFMAs will want them, all done some time before the barrier that waits for them.
    auto kstep = [&](auto buf_c, auto fresh_c, int cs, int rd_stage) __attribute__((always_inline)) {
        constexpr int BUF = decltype(buf_c)::value;
        constexpr bool FRESH = decltype(fresh_c)::value;
        const typename CODES::Sums zero = {0, 0, 0, 0};
        const uint8_t *const wp = smem + rd_stage + w_lane, *const xp = smem + rd_stage + x_lane;
        e_static_for<NM>([&](auto t_c) __attribute__((always_inline)) {
            constexpr int t = decltype(t_c)::value, j = t / TM, i = t % TM;
            acc[j][i] = CODES::multiply(F[BUF][j], F[BUF][TN + i], FRESH ? zero : acc[j][i]);
            e_static_for<MOVES>([&](auto n_c) __attribute__((always_inline)) {
                constexpr int n = decltype(n_c)::value;
                if constexpr (1 + n * (NM * 3 / 4) / MOVES == t) issue_transfer(n_c, cs);
            });
            e_static_for<2 * NF>([&](auto o_c) __attribute__((always_inline)) {
                constexpr int o = decltype(o_c)::value, fo = o / 2;     // fo-th fragment in order of first use: W0, all X, other W
                constexpr int f = (fo == 0) ? 0 : (fo <= TM ? TN + fo - 1 : fo - TM);
                if constexpr (o * (NM - 8) / (2 * NF) == t) {
                    if constexpr (o % 2 == 0) read_lo(std::integral_constant<int, BUF ^ 1>{}, f, wp, xp);
                    else read_hi(std::integral_constant<int, BUF ^ 1>{}, f, wp, xp);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using BT = std::true_type;
    using BF = std::false_type;

    // ---- prologue of the whole stream.  K-step p of the stream lives in ring stage p % STAGES
    if (bias == nullptr) {
        for (int b = 0; b < C::SC_BUFFERS; ++b)
            for (int i = tid; i < C::BN / 2; i += C::THREADS)
                reinterpret_cast<uint32_t *>(sc_all + b * C::SC_BYTES + C::BM * 4 + C::BN * 4)[i] = 0u;
    }
    set_tile_pointers(first_tile);
    if constexpr (C::SC_BUFFERS == 2) issue_scales(first_tile, 0);
    for (int s = 0; s < C::STAGES; ++s) {
        e_static_for<MOVES>([&](auto n_c) __attribute__((always_inline)) { issue_transfer(n_c, s * C::STAGE_BYTES); });
        advance_cursor();
    }
    e_wait_vmcnt<(C::STAGES - 1) * MOVES>();
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        read_lo(I0{}, f, smem + w_lane, smem + x_lane);
        read_hi(I0{}, f, smem + w_lane, smem + x_lane);
    }

    int cs = 0, sb = 0;                                   // ring stage of the K-step being computed, scale buffer of the current tile
    for (int tile = first_tile; tile < tile_end; tile += slots) {
        // K-step p of the stream: once at most the transfers of STAGES - 2 later ones of this wave are outstanding, p + 1 has landed for it; after the
        // barrier it has landed for every wave, and every wave has the fragments of p in registers (the barrier waits for their reads): stage cs is refilled
        auto step = [&](auto buf_c, auto fresh_c) __attribute__((always_inline)) {
            constexpr bool FRESH = decltype(fresh_c)::value;
            e_wait_vmcnt<(C::STAGES - 2) * MOVES>();
            __syncthreads();
            if constexpr (FRESH) {
                // with one buffer: the tile's own, now that all waves are past the epilogue before
                int ts = C::SC_BUFFERS == 2 ? tile + slots : tile;
                if (ts < tile_end) {
                    asm volatile("" : "+s"(ts));
                    issue_scales(ts, C::SC_BUFFERS == 2 ? sb ^ 1 : 0);
                }
            }
            const int ns = cs == (C::STAGES - 1) * C::STAGE_BYTES ? 0 : cs + C::STAGE_BYTES;
            kstep(buf_c, fresh_c, cs, ns);
            advance_cursor();
            cs = ns;
        };
        step(I0{}, BT{});
        int left = ksteps - 1;
        for (; left >= 2; left -= 2) {
            step(I1{}, BF{});
            step(I0{}, BF{});
        }
        // its LDS reads fetch the first fragments of the block's next tile: they live through the epilogue
        if (left == 1) {
            step(I1{}, BF{});
        } else {                                                 // an odd number of K-steps (no K that calls have): they are in the other buffer.  Without this
#pragma unroll                                                   // branch the compiler moves accumulators about in the loop, and the affine kernels use scratch memory
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int e = 0; e < CODES::REGS; ++e) F[0][f][e] = F[1][f][e];
        }

        // ---- epilogue.  16x16 result layout: lane (c, q) holds column c = token and rows 4 q + r = channels
        const int tm = tile / tiles_n, tn = tile % tiles_n;
        const int row0 = tm * C::BM + wm * TM * 16, col0 = tn * C::BN + wn * TN * 16;
        const uint8_t *sc = sc_all + sb * C::SC_BYTES;
        const float *scx = reinterpret_cast<const float *>(sc) + wm * TM * 16 + c;
        const float *scw = reinterpret_cast<const float *>(sc + C::BM * 4) + wn * TN * 16 + 4 * q;
        const uint16_t *scb = reinterpret_cast<const uint16_t *>(sc + C::BM * 4 + C::BN * 4) + wn * TN * 16 + 4 * q;
        const float *scz = reinterpret_cast<const float *>(sc + C::SC_SYM_BYTES) + wm * TM * 16 + c;
        const float *scs = reinterpret_cast<const float *>(sc + C::SC_SYM_BYTES + C::BM * 4) + wn * TN * 16 + 4 * q;
        const int rows_left = M - row0, cols_left = N - col0;
        float sxm[TM], rz[SHIFTED ? TM : 1];
#pragma unroll
        for (int i = 0; i < TM; ++i) sxm[i] = scx[i * 16];
        if constexpr (SHIFTED) {
#pragma unroll
            for (int i = 0; i < TM; ++i) rz[i] = 7.5f - scz[i * 16];
        }
        uint8_t *ep = smem + C::STAGES * C::STAGE_BYTES + C::SC_BUFFERS * C::SC_BYTES + wave * (16 * C::EP_PITCH);
        const int rd_row = lane >> 3, rd_col = lane & 7;
        v4i rowv[2];
        // rows of piece (i, jp) as they come back from LDS: 8 tokens x 128 bytes a store
        auto store_piece = [&](int i, int jp) {
            uint16_t *yp = Y + (size_t)(row0 + i * 16 + rd_row) * N + col0 + jp * 64 + rd_col * 8;
            auto store = [&](int it) {
                v4i *const dst = reinterpret_cast<v4i *>(yp + (size_t)it * 8 * N);
                if constexpr (STREAM_Y) __builtin_nontemporal_store(rowv[it], dst);
                else *dst = rowv[it];
            };
            if (rows_left - i * 16 >= 16 && cols_left - jp * 64 >= 64) {
#pragma unroll
                for (int it = 0; it < 2; ++it) store(it);
            } else {
#pragma unroll
                for (int it = 0; it < 2; ++it)
                    if (rd_col * 8 < cols_left - jp * 64 && rd_row < rows_left - (i * 16 + it * 8)) store(it);
            }
        };
#pragma unroll
        for (int jp = 0; jp < TN / 4; ++jp) {
            float4 swq[4], bq[4], wsq[SHIFTED ? 4 : 1];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                swq[jj] = *reinterpret_cast<const float4 *>(scw + (4 * jp + jj) * 16);
                if constexpr (SHIFTED) wsq[jj] = *reinterpret_cast<const float4 *>(scs + (4 * jp + jj) * 16);
                const uint2 b = *reinterpret_cast<const uint2 *>(scb + (4 * jp + jj) * 16);
                bq[jj] = make_float4(__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xFFFF0000u), __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xFFFF0000u));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                uint2 out[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    typename CODES::Sum r0, r1, r2, r3;
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r0) : "a"(acc[4 * jp + jj][i][0]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r1) : "a"(acc[4 * jp + jj][i][1]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r2) : "a"(acc[4 * jp + jj][i][2]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r3) : "a"(acc[4 * jp + jj][i][3]));
                    float a0 = CODES::sum(r0), a1 = CODES::sum(r1), a2 = CODES::sum(r2), a3 = CODES::sum(r3);
                    if constexpr (SHIFTED) {
                        a0 = fmaf(rz[i], wsq[jj].x, a0); a1 = fmaf(rz[i], wsq[jj].y, a1);
                        a2 = fmaf(rz[i], wsq[jj].z, a2); a3 = fmaf(rz[i], wsq[jj].w, a3);
                    }
                    const float y0 = fmaf(a0, swq[jj].x * sxm[i], bq[jj].x), y1 = fmaf(a1, swq[jj].y * sxm[i], bq[jj].y);
                    const float y2 = fmaf(a2, swq[jj].z * sxm[i], bq[jj].z), y3 = fmaf(a3, swq[jj].w * sxm[i], bq[jj].w);
                    out[jj] = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
                    if constexpr (DEBUG) {
                        const int m = row0 + i * 16 + c, n = col0 + (4 * jp + jj) * 16 + 4 * q;
                        if (m < M && n < N) *reinterpret_cast<int4 *>(acc_debug + (size_t)m * N + n) = make_int4((int)a0, (int)a1, (int)a2, (int)a3);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (i > 0) store_piece(i - 1, jp);
                else if (jp > 0) store_piece(TM - 1, jp - 1);
                __builtin_amdgcn_sched_barrier(0);
                lanes_exchange_fence();
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) *reinterpret_cast<uint2 *>(ep + c * C::EP_PITCH + (jj * 16 + 4 * q) * 2) = out[jj];
                lanes_exchange_fence();
#pragma unroll
                for (int it = 0; it < 2; ++it) rowv[it] = *reinterpret_cast<const v4i *>(ep + (it * 8 + rd_row) * C::EP_PITCH + rd_col * 16);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        store_piece(TM - 1, TN / 4 - 1);
        if constexpr (C::SC_BUFFERS == 2) sb ^= 1;
    }
    e_wait_vmcnt<0>();      // transfers issued past the last tile must not outlive the block's LDS allocation
}

}  // namespace qvggt
