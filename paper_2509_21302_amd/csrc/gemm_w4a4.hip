// Online kernel 2: int4 x int4 GEMM with int32 accumulation on the int8 matrix cores and a
// fused dequantise + bias epilogue (paper Sec. 3.2, granularity paragraph: the scales are
// constant along the summed dimension, so the sum stays in integers and is rescaled once).
//
//   acc[t, o] = sum_j Xq[t, j] * Wq[o, j]
//   Y[t, o]   = bf16( acc[t, o] * sx[t] * sw[o] + bias[o] )
//
// Data movement.  A block owns a tile of BM tokens x BN channels and walks over many such
// tiles (persistent grid).  The packed codes of both operands travel from global memory
// straight into LDS (global_load_lds_dwordx4: no staging registers, no LDS store
// instructions) in K-tiles of 64 bytes = 128 codes per row, through a ring of STAGES
// buffers; the K-tiles of successive output tiles form one continuous stream, so the first
// K-tiles of the next output tile are in flight while the current one finishes.
//
// LDS layout of a stage: rows of 64 bytes (BM token rows, then BN channel rows); the four
// 16-byte chunks of a row are XOR-swizzled with bits 2..3 of the row index.  The transfer
// writes 1 KiB contiguous per wavefront instruction (16 rows); the swizzle is applied on the
// global side (which chunk a lane fetches).  A fragment read is one ds_read_b128 per lane:
// lane (row = lane % 32, half = lane / 32) takes chunk 2*pair + half of its row, i.e. its 8
// bytes of K-step 2*pair and its 8 bytes of K-step 2*pair + 1.  Any 16 consecutive rows hit the
// 16 distinct 16-byte groups of the 64 LDS banks, so these reads are conflict free.  The order in
// which codes meet inside a K-step is the same for both operands, which is all a dot
// product needs.
//
// Arithmetic.  A wavefront expands packed bytes to int8 in registers right before the MFMA:
// each code is kept in the HIGH nibble of its byte (v & 0xF0F0F0F0 for the odd codes,
// (v << 4) & 0xF0F0F0F0 for the even ones), i.e. as 16 * code with the sign in place, so no
// sign extension is needed.  Both operands are expanded the same way, hence the accumulator
// is exactly 256 * acc (|256 * acc| <= 256 * 64 * 8192 = 2^27) and the factor is removed
// exactly afterwards.  The weights are the MFMA row operand and the activations its column
// operand, so a lane ends up with 4 consecutive output channels of one token.
//
// Epilogue.  Accumulators stay in AGPRs; each 32x64 piece is scaled, rounded to bf16 and turned into rows through a
// small wave-private LDS tile, so that every store instruction writes whole 128-byte lines.  They are streaming
// (non-temporal) stores: Y is not read again here, and kept out of L2 it leaves the weights resident there.
//
// Schedule.  A K-step of a wavefront is TM*TN MFMAs (32x32x32 int8); the LDS reads of the
// next pair of K-steps and the expansion of the next K-step's fragments are dealt out one
// piece per MFMA, fenced so that the compiler keeps the interleave: the vector ALU and LDS
// work runs in the shadow of the matrix pipe.
#include "gemm_plan.h"
#include "gemm_tiles256.h"
#include "lds_transfer.h"
#include "qvggt_common.h"
#include "resident.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace qvggt {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

namespace {

constexpr int KT_BYTES = 64;       // packed bytes per row per K-tile: 128 codes = 4 MFMA K-steps = 2 pairs

// TM x TN: 32x32 sub-tiles per wave along tokens / channels; WM x WN: waves per block; STAGES: LDS ring depth
// ASYM: the per-tile scale area also carries the tokens' zero points and the channels' weight code sums
template <int TM, int TN, int WM, int WN, int STAGES, bool ASYM = false>
struct StreamCfg {
    static constexpr int NW = WM * WN, THREADS = NW * 64;
    static constexpr int BM = WM * TM * 32, BN = WN * TN * 32, ROWS = BM + BN;
    static constexpr int STAGE_BYTES = ROWS * KT_BYTES;
    static constexpr int GROUPS = ROWS / 16;            // 16-row groups: one wave-wide transfer instruction each
    static constexpr int LPW = GROUPS / NW;             // transfers per wave per K-tile
    static constexpr int NM = TM * TN, NF = TM + TN;
    static constexpr int SC_SYM_BYTES = BM * 4 + BN * 4 + BN * 2;   // per tile: sx f32, sw f32, bias bf16 (as in memory)
    static constexpr int SC_SYM_GROUPS = BM / 64 + BN / 64 + BN / 128;
    static constexpr int SC_BYTES = SC_SYM_BYTES + (ASYM ? BM * 4 + BN * 4 : 0);        // then zero points f32, code sums f32
    static constexpr int SC_GROUPS = SC_SYM_GROUPS + (ASYM ? BM / 64 + BN / 64 : 0);
    static constexpr int EP_PITCH = 128 + 16;           // bytes per token row of a wave's epilogue staging tile (64 channels + pad)
    static constexpr int EP_BYTES = NW * 32 * EP_PITCH;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + 2 * SC_BYTES + EP_BYTES;
    // A tile's scales are sent for during the first K-tile of the tile before, and 2 ktiles - 1 K-tiles' transfers follow before the last wait
    // ahead of their use, which lets STAGES - 3 K-tiles' be outstanding: with fewer K-tiles it would not cover them
    static constexpr int MIN_KTILES = (STAGES - 1) / 2;
    static_assert(TN % 2 == 0, "the epilogue handles channel sub-tiles in pairs");
    static_assert(GROUPS % NW == 0, "16-row groups do not divide among the waves");
    static_assert(BM % 128 == 0 && BN % 128 == 0, "scale transfers assume multiples of 128");
    static_assert(STAGES >= 3, "ring needs one stage being read, one landed, one in flight");
};

// one packed dword (8 codes) -> two dwords of int8: codes 1,3,5,7 and codes 0,2,4,6, each as 16 * code
#define QVGGT_EXPAND_HALF(p, dst, k)                                   \
    do {                                                               \
        const uint32_t p_ = (uint32_t)(p);                             \
        (dst)[(k)] = (int)(p_ & 0xF0F0F0F0u);                          \
        (dst)[(k) + 1] = (int)((p_ << 4) & 0xF0F0F0F0u);               \
    } while (0)

// a pointer that is the same in all lanes, in scalar registers (the transfers' base operand has to be; the compiler does not always see it)
__device__ inline const uint8_t *scalar_pointer(const uint8_t *p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
}
template <class F, int... Is>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <int N, class F>
__device__ inline void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
template <int N>
__device__ inline void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace

// CB: bits a stored code occupies: 4 (two codes per byte, expanded in registers) or 8 (int8 codes, fed to the MFMA as read)
// ASYM: activations carry affine codes u with a zero point per token, stored as u - 8 (Xq) and zp (xzero); the epilogue adds
// (8 - zp[t]) * wsum[o] (wsum[o] = sum_j qw[o, j], exact in fp32) to the accumulator before the scales
// BLK (int8 codes): the operands are "int8 blocks": rows grouped in blocks of 128 with the K-tiles outermost, K-tile kt of row r at
// ((r / 128) * (K / 64) + kt) * 8192 + (r % 128) * 64, its four 16-byte chunks already in the swizzled order of the LDS stage, so
// that what a wave fetches of a K-tile is 8 KiB (4 KiB in the small configuration) contiguous in memory
// LAST_FIRST: the highest-numbered blocks of every XCD take the first tiles (the ones that a preceding set of tiles in the same launch
// left without a last one)
template <int TM, int TN, int WM, int WN, int STAGES, int CB, bool DEBUG, bool ASYM, bool BLK, bool LAST_FIRST = false>
__device__ __forceinline__ void w4a4_tiles(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int N, int K,
    uint16_t *__restrict__ Y, int32_t *__restrict__ acc_debug, const float *__restrict__ xzero, const float *__restrict__ wsum)
{
    // the dynamic segment by its own name: handed in as a pointer it costs registers in the address arithmetic, and the affine small kernel
    // had none left (8 bytes of scratch, 32 x 256 -> 2784 5.7 -> 5.95 us)
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    using C = StreamCfg<TM, TN, WM, WN, STAGES, ASYM>;
    constexpr int NM = C::NM, NF = C::NF, LPW = C::LPW;
    constexpr int DMA_SHIFT = (LPW > 4) ? 4096 : 0;             // keeps the transfers' instruction offsets inside [-4096, 4095]
    static_assert(LPW <= 8, "instruction offsets of a wave's transfers must fit 13 signed bits");
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    uint8_t *sc_all = smem + STAGES * C::STAGE_BYTES;           // two buffers of SC_BYTES
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;            // LDS byte address of the dynamic segment

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    static_assert(CB == 4 || CB == 8, "codes are stored in 4 or 8 bits");
    static_assert(!BLK || CB == 8, "the blocked operand format holds int8 codes");
    constexpr int KSTEPS = (CB == 4) ? 4 : 2;                   // MFMA K-steps (32 codes each) in a K-tile of 64 bytes per row
    const int KB = (CB == 4) ? (K >> 1) : K;                    // bytes per row of codes
    const int ktiles = KB / KT_BYTES;
    const int ntiles = tiles_m * tiles_n;

    // Tile assignment: workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  XCD x owns the
    // contiguous tile range [x * per_xcd, (x + 1) * per_xcd) (channel tiles fastest), its blocks take them in turn.
    const int per_xcd = (ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7, slots = gridDim.x >> 3, slot = LAST_FIRST ? slots - 1 - (int)(blockIdx.x >> 3) : (int)(blockIdx.x >> 3);
    const int tile_end = min((xcd + 1) * per_xcd, ntiles);
    const int first_tile = xcd * per_xcd + slot;
    if (first_tile >= tile_end) return;
    const int last_tile = tile_end - 1 - ((tile_end - 1 - first_tile) % slots);   // this block's last tile

    // ---- global -> LDS transfers.  Lane l of a transfer covers row l / 4 of a 16-row group and lands in 16-byte
    // slot l % 4 of that row; it fetches the chunk that the swizzle puts there.
    const int t_row = lane >> 2;
    const int t_chunk = (lane & 3) ^ ((t_row >> 2) & 3);
    // A wave's LPW groups lie in one operand (X rows come first in a stage), so all its transfers share one base.
    static_assert((C::BM / 16) % LPW == 0, "a wave's 16-row groups must not straddle the two operands");
    constexpr uint32_t BASE_SHIFT = 4096;                       // keeps the pre-compensated lane offsets non-negative
    const bool loads_x = wave * LPW * 16 < C::BM;
    uint32_t lane_off[LPW];
    const uint8_t *tile_base;                                   // wave-uniform: row 0 of the operand's tile, minus BASE_SHIFT
    int ld_tile = first_tile, ld_kt = 0, ld_stage = 0;
    static_assert(!BLK || 8192 % (LPW * 1024) == 0, "a wave's transfers of a K-tile must lie inside one 128-row block");
    if constexpr (BLK) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) lane_off[i] = (i * 64 + lane) * 16 + BASE_SHIFT - (i * 1024 - DMA_SHIFT);
    }
    auto set_tile_pointers = [&](int t) {
        const int tm = t / tiles_n, tn = t % tiles_n;
        const int row0 = loads_x ? tm * C::BM : tn * C::BN;     // first row of the tile in its operand
        if constexpr (BLK) {
            const int row = row0 + wave * LPW * 16 - (loads_x ? 0 : C::BM);          // first row of this wave's share
            const int blk = min(row / 128, ((loads_x ? M : N) + 127) / 128 - 1);        // past the end: re-read the last block (unused)
            tile_base = scalar_pointer((loads_x ? Xq : Wq) + (size_t)blk * ktiles * 8192 + (row % 128) * KT_BYTES - BASE_SHIFT);
            return;
        }
        const int last = (loads_x ? M : N) - 1 - row0;          // last existing row, relative to row0 (>= 0)
        tile_base = scalar_pointer((loads_x ? Xq : Wq) + (size_t)row0 * KB - BASE_SHIFT);
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int r = (wave * LPW + i) * 16 + t_row - (loads_x ? 0 : C::BM);   // row inside the operand's tile
            lane_off[i] = (uint32_t)min(r, last) * (uint32_t)KB + t_chunk * 16 + BASE_SHIFT - (i * 1024 - DMA_SHIFT);
        }
    };
    // The K-tile under the load cursor goes to ring stage ld_stage, one transfer instruction at a time (a wave that issues
    // them back to back stalls on each: they are dealt out between MFMAs instead); then the cursor moves on, across
    // output tiles (past this block's last tile it re-reads that tile: never used, keeps the transfers in flight uniform).
    auto issue_transfer = [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        const uint8_t *base = tile_base + (BLK ? (size_t)ld_kt * 8192 : (size_t)ld_kt * KT_BYTES);
        // the wave's LPW KiB of a stage are contiguous; the LDS base points DMA_SHIFT into them
        dma16<i * 1024 - DMA_SHIFT>(lane_off[i], base, lds0 + ld_stage * C::STAGE_BYTES + wave * LPW * 1024 + DMA_SHIFT);
    };
    auto advance_cursor = [&]() {
        ld_stage = (ld_stage + 1 == STAGES) ? 0 : ld_stage + 1;
        if (++ld_kt == ktiles) {
            ld_kt = 0;
            ld_tile = min(ld_tile + slots, last_tile);
            set_tile_pointers(ld_tile);
        }
    };
    auto issue_ktile = [&]() {
        static_for<LPW>([&](auto i_c) { issue_transfer(i_c); });
        advance_cursor();
    };
    // per-tile scales to LDS buffer sb, as they are in memory: sx of the tile's tokens, sw and bias of its channels
    auto issue_scales = [&](int t, int sb) {
        const int tm = t / tiles_n, tn = t % tiles_n;
        const uint32_t dst = lds0 + STAGES * C::STAGE_BYTES + sb * C::SC_BYTES;
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
                    dma4(reinterpret_cast<const uint32_t *>(bias) + min(tn * (C::BN / 2) + h * 64 + lane, N / 2 - 1),
                         dst + C::BM * 4 + C::BN * 4 + h * 256);
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

    // ---- fragments
    v16i acc[TN][TM];   // [channel sub-tile j][token sub-tile i]
    v4i raw[NF];        // packed fragments of a pair of K-steps: W sub-tiles, then X sub-tiles
    v4i F[2][NF];       // expanded fragments of one K-step: [K-step parity][W sub-tiles, then X sub-tiles]
    const int frow = lane & 31, fhalf = lane >> 5;
    const int fsw = (frow >> 2) & 3;
    // byte offsets inside a stage of this lane's chunk of pair 0; pair 1 is the same with chunk bit 1 (byte bit 5) flipped
    const int w_off = (C::BM + wn * TN * 32 + frow) * KT_BYTES + ((fhalf ^ fsw) << 4);
    const int x_off = (wm * TM * 32 + frow) * KT_BYTES + ((fhalf ^ fsw) << 4);
    auto read_frag = [&](int f, int stage, int pair) {
        const int off = ((f < TN) ? w_off : x_off) ^ (pair << 5);
        raw[f] = *reinterpret_cast<const v4i *>(smem + stage * C::STAGE_BYTES + off + ((f < TN) ? f : f - TN) * 32 * KT_BYTES);
    };
    // One K-step: NM slots of {one MFMA, a share of the side work}.  The side work is the expansion of the NEXT K-step's
    // fragments, a dword (3 ALU ops) at a time, evenly over the slots:
    //   PAR == 0 (first K-step of a pair):  raw[f].zw -> F[1][f].  Once both dwords of raw[f] are used it is dead, and the
    //             read of the next pair's fragment f (ring stage rd_stage, pair rd_pair) is issued into it in the next slot;
    //   PAR == 1 (second K-step of a pair): raw[f].xy -> F[0][f]; slot 0 issues the reads that did not fit into the step before.
    // So a fragment's LDS read is issued most of a K-step before its first use, and reads are spread over the K-step.
    auto kstep = [&](auto step_c, auto fresh_c, int rd_stage, int rd_pair) {
        constexpr int STEP = decltype(step_c)::value, PAR = STEP & 1;   // STEP: K-step inside the K-tile
        constexpr bool FRESH = decltype(fresh_c)::value;
        const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        static_for<NM>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value, j = t / TM, i = t % TM;
            acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(F[PAR][j], F[PAR][TN + i], FRESH ? zero : acc[j][i], 0, 0, 0);
            // this K-tile's share of the global -> LDS transfers: transfer n goes out in slot (2n + 1) * KSTEPS * NM / (2 * LPW) of the K-tile
            static_for<LPW>([&](auto n_c) {
                constexpr int n = decltype(n_c)::value;
                if constexpr ((2 * n + 1) * KSTEPS * NM / (2 * LPW) == STEP * NM + t) issue_transfer(n_c);
            });
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int done = ((2 * f + 2) * NM + 2 * NF - 1) / (2 * NF) - 1;   // slot of the PAR == 0 step that uses raw[f] last
                if (PAR == 0 ? (done + 1 == t) : (t == 0 && done + 1 >= NM)) read_frag(f, rd_stage, rd_pair);
            }
#pragma unroll
            for (int h = t * 2 * NF / NM; h < (t + 1) * 2 * NF / NM; ++h) {
                if (PAR == 0) QVGGT_EXPAND_HALF(raw[h >> 1][2 + (h & 1)], F[1][h >> 1], 2 * (h & 1));
                else QVGGT_EXPAND_HALF(raw[h >> 1][h & 1], F[0][h >> 1], 2 * (h & 1));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // One K-step on int8 codes: a lane's 16 bytes of a fragment are the MFMA operand as they are, so F[STEP] is filled
    // straight from LDS.  While K-step STEP runs on F[STEP], the fragments of the next K-step (ring stage rd_stage, K-step
    // rd_step of that K-tile) are read into F[STEP ^ 1], one every NM / NF slots, in the order the MFMAs will want them.
    auto kstep8 = [&](auto step_c, auto fresh_c, int rd_stage, int rd_step) {
        constexpr int STEP = decltype(step_c)::value;
        constexpr bool FRESH = decltype(fresh_c)::value;
        const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        static_for<NM>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value, j = t / TM, i = t % TM;
            acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(F[STEP][j], F[STEP][TN + i], FRESH ? zero : acc[j][i], 0, 0, 0);
            static_for<LPW>([&](auto n_c) {
                constexpr int n = decltype(n_c)::value;
                if constexpr ((2 * n + 1) * KSTEPS * NM / (2 * LPW) == STEP * NM + t) issue_transfer(n_c);
            });
            static_for<NF>([&](auto o_c) {
                constexpr int o = decltype(o_c)::value;                  // o-th read: W0, all X, then the other W
                constexpr int f = (o == 0) ? 0 : (o <= TM ? TN + o - 1 : o - TM);
                if constexpr (o * NM / NF == t) {
                    const int off = ((f < TN) ? w_off : x_off) ^ (rd_step << 5);
                    F[STEP ^ 1][f] = *reinterpret_cast<const v4i *>(smem + rd_stage * C::STAGE_BYTES + off + ((f < TN) ? f : f - TN) * 32 * KT_BYTES);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using BT = std::true_type;
    using BF = std::false_type;

    // ---- prologue of the whole stream
    if (bias == nullptr) {      // no bias: both bias areas stay zero for the whole kernel
        for (int b = 0; b < 2; ++b)
            for (int i = tid; i < C::BN / 2; i += C::THREADS)
                reinterpret_cast<uint32_t *>(sc_all + b * C::SC_BYTES + C::BM * 4 + C::BN * 4)[i] = 0u;
    }
    set_tile_pointers(first_tile);
    issue_scales(first_tile, 0);
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue_ktile();
    wait_vmcnt<(STAGES - 2) * LPW>();
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) read_frag(f, 0, 0);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        if constexpr (CB == 4) {
            QVGGT_EXPAND_HALF(raw[f][0], F[0][f], 0);
            QVGGT_EXPAND_HALF(raw[f][1], F[0][f], 2);
        } else {
            F[0][f] = raw[f];
        }
    }

    const int c = lane & 31, g = lane >> 5;

    int cs = 0, sb = 0;                                   // ring stage being computed on, scale buffer of the current tile
    for (int tile = first_tile; tile < tile_end; tile += slots) {
        // one K-tile of the stream: four K-steps on ring stage cs.  The first K-tile of an output tile starts the
        // accumulators from zero (FRESH) and sends for the scales of the block's next output tile.
        auto ktile = [&](auto fresh_c) {
            constexpr bool FRESH = decltype(fresh_c)::value;
            // K-tile q+1 of the stream has landed for this wave once at most (STAGES-3) later K-tiles are outstanding; after
            // the barrier it has landed for every wave, and every wave is done reading K-tile q-1, whose stage is reused.
            wait_vmcnt<(STAGES - 3) * LPW>();
            __syncthreads();
            if (FRESH && tile + slots < tile_end) {
                int tnext = tile + slots;
                asm volatile("" : "+s"(tnext));             // keeps the address arithmetic of the scale transfers inside this branch
                issue_scales(tnext, sb ^ 1);
            }
            const int ns = (cs + 1 == STAGES) ? 0 : cs + 1;
            if constexpr (CB == 4) {
                kstep(I0{}, fresh_c, cs, 1);
                kstep(I1{}, BF{}, cs, 1);
                kstep(I2{}, BF{}, ns, 0);
                kstep(I3{}, BF{}, ns, 0);
            } else {
                kstep8(I0{}, fresh_c, cs, 1);
                kstep8(I1{}, BF{}, ns, 0);
            }
            advance_cursor();
            cs = ns;
        };
        ktile(BT{});
        for (int kt = 1; kt < ktiles; ++kt) ktile(BF{});

        // ---- epilogue.  32x32 result layout: lane l holds column (l % 32) = token and rows 8*(r/4) + 4*(l/32) + r%4 = channels,
        // i.e. per register quad q four consecutive channels 8q + 4*(l/32) + 0..3.  Scale + bias + bf16 in registers.
        const int tm = tile / tiles_n, tn = tile % tiles_n;
        const int row0 = tm * C::BM + wm * TM * 32, col0 = tn * C::BN + wn * TN * 32;   // first token / channel of this wave
        const uint8_t *sc = sc_all + sb * C::SC_BYTES;
        const float *scx = reinterpret_cast<const float *>(sc);
        const float *scw = reinterpret_cast<const float *>(sc + C::BM * 4) + wn * TN * 32 + 4 * g;
        const uint16_t *scb = reinterpret_cast<const uint16_t *>(sc + C::BM * 4 + C::BN * 4) + wn * TN * 32 + 4 * g;
        const int rows_left = M - row0;                      // tokens of this wave's rows that exist
        const int cols_left = N - col0;                      // channels of this wave's columns that exist (a multiple of 16)
        float sxm[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) sxm[i] = scx[(wm * TM + i) * 32 + c] * (CB == 4 ? 1.0f / 256.0f : 1.0f);
        // affine activation codes: (8 - zp) of this lane's tokens, in the accumulator's units (256 per unit for packed codes)
        const float *scz = reinterpret_cast<const float *>(sc + C::SC_SYM_BYTES);
        const float *scs = reinterpret_cast<const float *>(sc + C::SC_SYM_BYTES + C::BM * 4) + wn * TN * 32 + 4 * g;
        float rz[ASYM ? TM : 1];
        if constexpr (ASYM) {
#pragma unroll
            for (int i = 0; i < TM; ++i) rz[i] = (8.0f - scz[(wm * TM + i) * 32 + c]) * (CB == 4 ? 256.0f : 1.0f);
        }
        {
            // A wave-private LDS tile [32 tokens][64 channels] turns the lane-per-token layout into rows, so
            // that a store instruction writes whole 128-byte lines (8 lanes x 16 bytes per token).  Whole lines can be
            // streamed past L2 (non-temporal) without write amplification, which leaves the weights resident there.
            uint8_t *ep = smem + STAGES * C::STAGE_BYTES + 2 * C::SC_BYTES + wave * (32 * C::EP_PITCH);
            const int rd_row = lane >> 3, rd_col = lane & 7;
#pragma unroll
            for (int jp = 0; jp < TN / 2; ++jp) {
                float4 swq[2][4], bq[2][4], wsq[ASYM ? 2 : 1][ASYM ? 4 : 1];
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        swq[jj][q] = *reinterpret_cast<const float4 *>(scw + (2 * jp + jj) * 32 + 8 * q);
                        if constexpr (ASYM) wsq[jj][q] = *reinterpret_cast<const float4 *>(scs + (2 * jp + jj) * 32 + 8 * q);
                        const uint2 b = *reinterpret_cast<const uint2 *>(scb + (2 * jp + jj) * 32 + 8 * q);
                        bq[jj][q] = make_float4(__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xFFFF0000u),
                                                __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xFFFF0000u));
                    }
                const bool col_ok = rd_col * 8 < cols_left - jp * 64;
                uint16_t *yp = Y + (size_t)(row0 + rd_row) * N + col0 + jp * 64 + rd_col * 8;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    // the token's scale folded into the channel scales once per piece: one multiply per channel instead of one per value
                    float4 sc[2][4];
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            sc[jj][q] = make_float4(swq[jj][q].x * sxm[i], swq[jj][q].y * sxm[i], swq[jj][q].z * sxm[i], swq[jj][q].w * sxm[i]);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            int a0, a1, a2, a3;
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a0) : "a"(acc[2 * jp + jj][i][4 * q]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a1) : "a"(acc[2 * jp + jj][i][4 * q + 1]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a2) : "a"(acc[2 * jp + jj][i][4 * q + 2]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a3) : "a"(acc[2 * jp + jj][i][4 * q + 3]));
                            float f0 = (float)a0, f1 = (float)a1, f2 = (float)a2, f3 = (float)a3;
                            if constexpr (ASYM) {      // integers below 2^27 that are multiples of 256 (packed codes), or below 2^24: exact
                                f0 = fmaf(rz[i], wsq[jj][q].x, f0); f1 = fmaf(rz[i], wsq[jj][q].y, f1);
                                f2 = fmaf(rz[i], wsq[jj][q].z, f2); f3 = fmaf(rz[i], wsq[jj][q].w, f3);
                            }
                            const float y0 = fmaf(f0, sc[jj][q].x, bq[jj][q].x), y1 = fmaf(f1, sc[jj][q].y, bq[jj][q].y);
                            const float y2 = fmaf(f2, sc[jj][q].z, bq[jj][q].z), y3 = fmaf(f3, sc[jj][q].w, bq[jj][q].w);
                            *reinterpret_cast<uint2 *>(ep + c * C::EP_PITCH + (jj * 32 + 8 * q + 4 * g) * 2) = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
                            if constexpr (DEBUG) {
                                const int m = row0 + i * 32 + c, n = col0 + (2 * jp + jj) * 32 + 8 * q + 4 * g;
                                if (m < M && n < N)
                                    *reinterpret_cast<int4 *>(acc_debug + (size_t)m * N + n) = make_int4(a0 >> (16 - 2 * CB), a1 >> (16 - 2 * CB), a2 >> (16 - 2 * CB), a3 >> (16 - 2 * CB));
                            }
                        }
                    __builtin_amdgcn_sched_barrier(0);
                    // the staging tile is private to the wave and LDS operations of a wave execute in order: no barrier instruction is
                    // needed, only the compiler has to be told that other lanes' writes are read next
                    lanes_exchange_fence();
                    // all four row groups are read before the first store: one LDS round trip per piece instead of four.  A piece
                    // that lies fully inside Y (the usual case, a wave-uniform test) stores without per-lane predicates.
                    v4i rowv[4];
#pragma unroll
                    for (int it = 0; it < 4; ++it) rowv[it] = *reinterpret_cast<const v4i *>(ep + (it * 8 + rd_row) * C::EP_PITCH + rd_col * 16);
                    if (rows_left - i * 32 >= 32 && cols_left - jp * 64 >= 64) {
#pragma unroll
                        for (int it = 0; it < 4; ++it) __builtin_nontemporal_store(rowv[it], reinterpret_cast<v4i *>(yp + (size_t)it * 8 * N));
                    } else {
#pragma unroll
                        for (int it = 0; it < 4; ++it)
                            if (col_ok && rd_row < rows_left - (i * 32 + it * 8)) __builtin_nontemporal_store(rowv[it], reinterpret_cast<v4i *>(yp + (size_t)it * 8 * N));
                    }
                    yp += (size_t)32 * N;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        sb ^= 1;
    }
    wait_vmcnt<0>();        // transfers issued past the last tile must not outlive the block's LDS allocation
}

template <int TM, int TN, int WM, int WN, int STAGES, int MINB, int CB, bool DEBUG, bool ASYM = false, bool BLK = false>
__global__ __launch_bounds__(WM * WN * 64, MINB) __attribute__((amdgpu_waves_per_eu(WM * WN * MINB / 4, WM * WN * MINB / 4))) void w4a4_gemm_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int N, int K,
    uint16_t *__restrict__ Y, int32_t *__restrict__ acc_debug, const float *__restrict__ xzero, const float *__restrict__ wsum)
{
    w4a4_tiles<TM, TN, WM, WN, STAGES, CB, DEBUG, ASYM, BLK>(Xq, sx, Wq, sw, bias, M, N, K, Y, acc_debug, xzero, wsum);
}

// int8 blocks in 256 x 256 tiles on the 16x16x64 instruction (gemm_tiles256.h): bound by the board's power and the way into LDS.  32976 x 4096 -> 1024 (two
// rounds of these tiles, the rest in the kernel below) 128 us with 32x32x32 products, 120 this way; the 8-bit MLP of 24 frames, both layers, with fc1 on the
// same instructions, 345 -> 328.
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void i8b_256_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int N, int K, uint16_t *__restrict__ Y, int tiles_m, int tiles_n)
{
    tiles256<Int8Tiles, false, false, true>(Xq, sx, Wq, sw, bias, M, N, K, Y, nullptr, tiles_m, tiles_n, nullptr, nullptr);
}

// The first `rows_main` token rows (a multiple of 256) in 256 x 256 tiles, which fill whole rounds of the chip, then the rest in 128 x 128
// tiles through a ring of twice the stages (the same LDS), in one launch: a block goes on to the rest when it is done, with no second
// launch behind the slowest block, and one block per compute unit has the LDS to keep seven K-tiles in flight, which is what a tile
// without company is bound by.
template <int CB, bool BLK, bool T256>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void w4a4_gemm_tail_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int rows_main, int N, int K, uint16_t *__restrict__ Y)
{
    if constexpr (T256) tiles256<Int8Tiles, false, false, true>(Xq, sx, Wq, sw, bias, rows_main, N, K, Y, nullptr, rows_main / 256, (N + 255) / 256, nullptr, nullptr);
    else w4a4_tiles<4, 4, 2, 2, 4, CB, false, false, BLK>(Xq, sx, Wq, sw, bias, rows_main, N, K, Y, nullptr, nullptr, nullptr);
    __syncthreads();                     // every wave is done with its LDS before the ring is laid out anew
    w4a4_tiles<2, 2, 2, 2, 8, CB, false, false, BLK, true>(Xq + (size_t)rows_main * (CB == 4 ? K / 2 : K), sx + rows_main, Wq, sw, bias,
                                                           M - rows_main, N, K, Y + (size_t)rows_main * N, nullptr, nullptr, nullptr);
}

// The same product for few tiles, as e2m3_gemm_few_kernel: the KW waves of a block divide K among themselves instead of the tile (wave w takes
// K-tiles w, w + KW, ...), fragments come from memory straight into registers, DEPTH K-tiles ahead, and the int32 partial sums meet in LDS at the
// end.  A tile of the streaming kernel that is alone on its compute unit is a serial chain of transfers, barriers, LDS reads and MFMAs along K.
template <int TM, int TN, int KW>
struct FewCfg {
    static constexpr int THREADS = KW * 64, BM = TM * 32, BN = TN * 32, NF = TM + TN;
    static constexpr int GROUPS = TM * TN * 4;              // of four accumulator registers of a lane
    static constexpr int PITCH = 64 * 16 + 128;             // bytes of a group and a gap: neighbouring groups start in different halves of the banks
    static constexpr int LDS_BYTES = KW * GROUPS * PITCH;
    static constexpr int OCTS = BN / 8, ITEMS = BM * OCTS;  // runs of eight channels of a token
    static_assert(128 % BM == 0 && 128 % BN == 0, "a tile lies in one block of the blocked operand format");
    static_assert(THREADS % OCTS == 0, "a thread's runs are the same channels of different tokens");
};

template <int TM, int TN, int KW, int DEPTH, int CB, bool ASYM, bool BLK>
__global__ __launch_bounds__(KW * 64, 1) void w4a4_gemm_few_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ sx, const uint8_t *__restrict__ Wq, const float *__restrict__ sw,
    const uint16_t *__restrict__ bias, int M, int N, int K, uint16_t *__restrict__ Y, int tiles_m, int tiles_n, bool tokens_first,
    const float *__restrict__ xzero, const float *__restrict__ wsum)
{
    using C = FewCfg<TM, TN, KW>;
    constexpr int NF = C::NF;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row_bytes = CB == 4 ? K / 2 : K, ktiles = row_bytes / KT_BYTES, ntiles = tiles_m * tiles_n;
    const int per_xcd = (ntiles + 7) >> 3;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= ntiles) return;
    const int fast = tokens_first ? tiles_m : tiles_n, outer = tile / fast, inner = tile - outer * fast;
    const int tm = tokens_first ? inner : outer, tn = tokens_first ? outer : inner;
    const int row0 = tm * C::BM, col0 = tn * C::BN;

    // fragments: W sub-tiles, then X sub-tiles.  A lane's 16 bytes are chunk 2 p + lane / 32 of its row's 64-byte K-tile (p = 0, 1)
    const int frow = lane & 31, fhalf = lane >> 5;
    const uint8_t *src[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const bool is_w = f < TN;
        const int first = is_w ? col0 + f * 32 : row0 + (f - TN) * 32;
        if constexpr (BLK) {
            src[f] = (is_w ? Wq : Xq) + (size_t)(first / 128) * ktiles * 8192 + ((first % 128) + frow) * 64 + ((fhalf ^ ((frow & 15) >> 2)) << 4);
        } else {                                            // rows past the operand's end: the last one (results unused)
            src[f] = (is_w ? Wq : Xq) + (size_t)min(first + frow, (is_w ? N : M) - 1) * row_bytes + fhalf * 16;
        }
    }
    // chunk 2 + lane / 32 of a K-tile, from chunk lane / 32: in blocks its slot differs in bit 1 (byte 32), to either side
    const int pair1 = BLK ? ((((fhalf ^ ((frow & 15) >> 2)) & 2) != 0) ? -32 : 32) : 32;
    const size_t kt_step = BLK ? 8192 : KT_BYTES;
    v4i F[DEPTH][NF][2];
    auto load = [&](auto d_c, int kt) {
        constexpr int d = decltype(d_c)::value;
        const size_t off = (size_t)min(kt, ktiles - 1) * kt_step;          // past the end: the last K-tile again (not used)
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            F[d][f][0] = *reinterpret_cast<const v4i *>(src[f] + off);
            F[d][f][1] = *reinterpret_cast<const v4i *>(src[f] + off + pair1);
        }
    };
    static_for<DEPTH>([&](auto d_c) { load(d_c, wave + decltype(d_c)::value * KW); });
    // what the epilogue needs, asked for before the products
    constexpr int IT = (C::ITEMS + C::THREADS - 1) / C::THREADS;
    const int oct = tid % C::OCTS, t0 = tid / C::OCTS, n = col0 + oct * 8;
    const int nc = min(n, N - 8);
    const float4 sw0 = *reinterpret_cast<const float4 *>(sw + nc), sw1 = *reinterpret_cast<const float4 *>(sw + nc + 4);
    uint4 bw = make_uint4(0u, 0u, 0u, 0u);
    if (bias != nullptr) bw = *reinterpret_cast<const uint4 *>(bias + nc);
    float4 ws0, ws1;
    if constexpr (ASYM) { ws0 = *reinterpret_cast<const float4 *>(wsum + nc); ws1 = *reinterpret_cast<const float4 *>(wsum + nc + 4); }
    float st[IT], zt[ASYM ? IT : 1];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int m = min(row0 + t0 + k * (C::THREADS / C::OCTS), M - 1);
        st[k] = sx[m] * (CB == 4 ? 1.0f / 256.0f : 1.0f);
        if constexpr (ASYM) zt[k] = (8.0f - xzero[m]) * (CB == 4 ? 256.0f : 1.0f);
    }
    v16i acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = 0;
    for (int kt = wave; kt < ktiles; kt += DEPTH * KW) {      // every condition is the same for the whole wave
        static_for<DEPTH>([&](auto d_c) {
            constexpr int d = decltype(d_c)::value;
            if (kt + d * KW < ktiles) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    // packed codes: the odd ones of the 32 in the high nibbles as they are, then the even ones moved there
                    constexpr int PARTS = CB == 4 ? 2 : 1;
#pragma unroll
                    for (int e = 0; e < PARTS; ++e) {
                        v4i op[NF];
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            if constexpr (CB == 4) op[f] = (e == 0 ? F[d][f][p] : F[d][f][p] << 4) & (int)0xF0F0F0F0;
                            else op[f] = F[d][f][p];
                        }
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int i = 0; i < TM; ++i) acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(op[j], op[TN + i], acc[j][i], 0, 0, 0);
                    }
                }
            }
            if (kt + DEPTH * KW < ktiles) load(d_c, kt + (d + DEPTH) * KW);
        });
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<int4 *>(smem + (wave * C::GROUPS + (j * TM + i) * 4 + q) * C::PITCH + lane * 16) =
                    make_int4(acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]);
    __syncthreads();
    // 32x32 result layout: group q of a sub-tile holds channels 8 q .. 8 q + 3 in lanes 0 .. 31 and 8 q + 4 .. 8 q + 7 in lanes 32 .. 63
    const float swv[8] = {sw0.x, sw0.y, sw0.z, sw0.w, sw1.x, sw1.y, sw1.z, sw1.w};
    const uint32_t bwv[4] = {bw.x, bw.y, bw.z, bw.w};
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int t = t0 + k * (C::THREADS / C::OCTS), m = row0 + t;
        if ((C::ITEMS % C::THREADS != 0 && t >= C::BM) || m >= M || n >= N) continue;
        const uint8_t *p = smem + ((oct / 4) * TM * 4 + (t / 32) * 4 + oct % 4) * C::PITCH + (t % 32) * 16;
        int a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < KW; ++w) {
            const int4 lo = *reinterpret_cast<const int4 *>(p + w * C::GROUPS * C::PITCH), hi = *reinterpret_cast<const int4 *>(p + w * C::GROUPS * C::PITCH + 512);
            a[0] += lo.x; a[1] += lo.y; a[2] += lo.z; a[3] += lo.w; a[4] += hi.x; a[5] += hi.y; a[6] += hi.z; a[7] += hi.w;
        }
        float fv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) fv[e] = (float)a[e];
        if constexpr (ASYM) {
            const float wsv[8] = {ws0.x, ws0.y, ws0.z, ws0.w, ws1.x, ws1.y, ws1.z, ws1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) fv[e] = fmaf(zt[k], wsv[e], fv[e]);
        }
        uint32_t out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[e] = pack_bf16x2(fmaf(fv[2 * e], swv[2 * e] * st[k], __uint_as_float(bwv[e] << 16)),
                                 fmaf(fv[2 * e + 1], swv[2 * e + 1] * st[k], __uint_as_float(bwv[e] & 0xFFFF0000u)));
        *reinterpret_cast<uint4 *>(Y + (size_t)m * N + n) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// every instantiation launched below, with the dynamic LDS it needs: packed codes (plain, accumulator dump, affine), int8 codes
// row-major and in blocks (plain, accumulator dump)
#define QVGGT_GEMM_KERNELS(TM, TN, WM, WN, ST, MB)                                                                                        \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 4, false, false, false>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES}, \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 4, true, false, false>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES},  \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 4, false, true, false>), StreamCfg<TM, TN, WM, WN, ST, true>::LDS_BYTES},   \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 8, false, false, false>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES}, \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 8, true, false, false>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES},  \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 8, false, false, true>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES},  \
    {reinterpret_cast<const void *>(w4a4_gemm_kernel<TM, TN, WM, WN, ST, MB, 8, true, false, true>), StreamCfg<TM, TN, WM, WN, ST, false>::LDS_BYTES}
#define QVGGT_FEW_KERNELS(TM, TN, KW, D)                                                                                                  \
    {reinterpret_cast<const void *>(w4a4_gemm_few_kernel<TM, TN, KW, D, 4, false, false>), FewCfg<TM, TN, KW>::LDS_BYTES}, \
    {reinterpret_cast<const void *>(w4a4_gemm_few_kernel<TM, TN, KW, D, 4, true, false>), FewCfg<TM, TN, KW>::LDS_BYTES},  \
    {reinterpret_cast<const void *>(w4a4_gemm_few_kernel<TM, TN, KW, D, 8, false, false>), FewCfg<TM, TN, KW>::LDS_BYTES}, \
    {reinterpret_cast<const void *>(w4a4_gemm_few_kernel<TM, TN, KW, D, 8, false, true>), FewCfg<TM, TN, KW>::LDS_BYTES}
static constexpr int TAIL_LDS_BYTES = std::max({StreamCfg<4, 4, 2, 2, 4>::LDS_BYTES, StreamCfg<2, 2, 2, 2, 8>::LDS_BYTES, Cfg256<Int8Tiles, false>::LDS_BYTES});
static const LdsKernel gemm_lds_kernel_list[] = {QVGGT_GEMM_KERNELS(4, 4, 2, 2, 4, 1), QVGGT_GEMM_KERNELS(2, 2, 2, 2, 3, 2),
                                                 {reinterpret_cast<const void *>(i8b_256_kernel), Cfg256<Int8Tiles, false>::LDS_BYTES},
                                                 QVGGT_GEMM_KERNELS(2, 2, 2, 2, 8, 1),
                                                 QVGGT_FEW_KERNELS(2, 2, 4, 2), QVGGT_FEW_KERNELS(1, 2, 4, 2), QVGGT_FEW_KERNELS(1, 1, 8, 2),
                                                 {reinterpret_cast<const void *>(w4a4_gemm_tail_kernel<4, false, false>), TAIL_LDS_BYTES},
                                                 {reinterpret_cast<const void *>(w4a4_gemm_tail_kernel<8, false, false>), TAIL_LDS_BYTES},
                                                 {reinterpret_cast<const void *>(w4a4_gemm_tail_kernel<8, true, false>), TAIL_LDS_BYTES},
                                                 {reinterpret_cast<const void *>(w4a4_gemm_tail_kernel<8, true, true>), TAIL_LDS_BYTES}};
#undef QVGGT_GEMM_KERNELS
#undef QVGGT_FEW_KERNELS
static const LdsKernels gemm_lds_kernels(gemm_lds_kernel_list);

template <int TM, int TN, int WM, int WN, int STAGES, int MINB, int CB, bool ASYM = false, bool BLK = false>
static hipError_t launch_gemm(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw, const void *bias,
                              int M, int N, int K, void *Y, int32_t *acc_debug, hipStream_t stream,
                              const float *xzero = nullptr, const float *wsum = nullptr)
{
    using C = StreamCfg<TM, TN, WM, WN, STAGES, ASYM>;
    // the variant that also writes the raw accumulators is a separate instantiation: the production kernel carries none of it
    const bool debug = acc_debug != nullptr;
    auto kern = w4a4_gemm_kernel<TM, TN, WM, WN, STAGES, MINB, CB, false, ASYM, BLK>;
    if constexpr (!ASYM) {
        if (debug) kern = w4a4_gemm_kernel<TM, TN, WM, WN, STAGES, MINB, CB, true, false, BLK>;
    } else {
        if (debug) return hipErrorInvalidValue;      // no accumulator dump with affine codes: the corrected sum is never an integer register
    }
    if ((CB == 4 ? K / 2 : K) / KT_BYTES < C::MIN_KTILES) return hipErrorInvalidValue;      // no plan asks for it
    hipError_t e = prepare_device();                 // the kernel's dynamic-LDS limit on this device (see gemm_lds_kernels above)
    if (e != hipSuccess) return e;
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    const int ntiles = tiles_m * tiles_n;
    int grid = 256 * MINB;                                // MINB resident blocks on each of the 256 compute units
    if (grid > (ntiles + 7) / 8 * 8) grid = (ntiles + 7) / 8 * 8;
    kern<<<grid, C::THREADS, C::LDS_BYTES, stream>>>(Xq, sx, Wq, sw, reinterpret_cast<const uint16_t *>(bias), M, N, K,
                                                     reinterpret_cast<uint16_t *>(Y), acc_debug, xzero, wsum);
    return hipGetLastError();
}

template <int CB, bool BLK>
static hipError_t launch_gemm_tail(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw, const void *bias, int M,
                                   int rows_main, int N, int K, void *Y, hipStream_t stream)
{
    if ((CB == 4 ? K / 2 : K) / KT_BYTES < StreamCfg<2, 2, 2, 2, 8>::MIN_KTILES) return hipErrorInvalidValue;      // no plan asks for it
    hipError_t e = prepare_device();
    if (e != hipSuccess) return e;
    auto kern = w4a4_gemm_tail_kernel<CB, BLK, BLK>;
    if constexpr (BLK) {
        if (!i8b_tiles256(rows_main, N, K)) kern = w4a4_gemm_tail_kernel<CB, BLK, false>;
    }
    kern<<<256, 256, TAIL_LDS_BYTES, stream>>>(Xq, sx, Wq, sw, reinterpret_cast<const uint16_t *>(bias), M, rows_main, N, K, reinterpret_cast<uint16_t *>(Y));
    return hipGetLastError();
}

static hipError_t launch_i8b_256(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw, const void *bias, int M, int N, int K, void *Y, hipStream_t stream)
{
    hipError_t e = prepare_device();
    if (e != hipSuccess) return e;
    const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
    i8b_256_kernel<<<std::min(256, (tiles_m * tiles_n + 7) / 8 * 8), 256, Cfg256<Int8Tiles, false>::LDS_BYTES, stream>>>(
        Xq, sx, Wq, sw, reinterpret_cast<const uint16_t *>(bias), M, N, K, reinterpret_cast<uint16_t *>(Y), tiles_m, tiles_n);
    return hipGetLastError();
}

template <int TM, int TN, int KW, int DEPTH, int CB, bool ASYM, bool BLK>
static hipError_t launch_gemm_few(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw, const void *bias, int M, int N, int K, void *Y,
                                  hipStream_t stream, const float *xzero, const float *wsum)
{
    using C = FewCfg<TM, TN, KW>;
    hipError_t e = prepare_device();
    if (e != hipSuccess) return e;
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    // neighbouring tiles of an XCD share tokens, or, where the weights are the larger operand and more than its L2 holds with anything else, channels
    const bool tokens_first = tiles_m < tiles_n && (long long)N * K * CB / 8 > (3 << 20);
    w4a4_gemm_few_kernel<TM, TN, KW, DEPTH, CB, ASYM, BLK><<<(tiles_m * tiles_n + 7) / 8 * 8, C::THREADS, C::LDS_BYTES, stream>>>(
        Xq, sx, Wq, sw, reinterpret_cast<const uint16_t *>(bias), M, N, K, reinterpret_cast<uint16_t *>(Y), tiles_m, tiles_n, tokens_first, xzero, wsum);
    return hipGetLastError();
}

// The tile shapes that the plan of gemm_plan.h names, over the token rows it gives them.
template <int CB, bool ASYM = false, bool BLK = false>
static hipError_t gemm_by_plan(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw, const void *bias,
                               int M, int N, int K, void *Y, int32_t *acc_debug, hipStream_t stream,
                               const float *xzero = nullptr, const float *wsum = nullptr)
{
#define QVGGT_ROWS(TM, TN, ST, MB, row0, rows)                                                                                           \
    launch_gemm<TM, TN, 2, 2, ST, MB, CB, ASYM, BLK>(Xq + (size_t)(row0) * (CB == 4 ? K / 2 : K), sx + (row0), Wq, sw, bias, rows, N, K, \
                                                     static_cast<uint16_t *>(Y) + (size_t)(row0) * N,                                    \
                                                     acc_debug ? acc_debug + (size_t)(row0) * N : nullptr, stream,                       \
                                                     ASYM ? xzero + (row0) : nullptr, wsum)
    if (acc_debug == nullptr) {                      // the dump is for the streaming kernel
#define QVGGT_FEW(TM, TN, KW, D) return launch_gemm_few<TM, TN, KW, D, CB, ASYM, BLK>(Xq, sx, Wq, sw, bias, M, N, K, Y, stream, xzero, wsum)
        switch (int8_instruction_few_tiles(M, N, K, CB, BLK)) {
            case FewTiles::kNone: break;
            case FewTiles::k64: QVGGT_FEW(2, 2, 4, 2);
            case FewTiles::k32x64: QVGGT_FEW(1, 2, 4, 2);
            case FewTiles::k32: QVGGT_FEW(1, 1, 8, 2);
        }
#undef QVGGT_FEW
    }
    const GemmPlan plan = int8_instruction_gemm_plan(M, N, K, CB, ASYM, acc_debug != nullptr);
    switch (plan.shape) {
        case GemmPlan::kBig:
            if constexpr (BLK) {
                if (acc_debug == nullptr && i8b_tiles256(M, N, K)) return launch_i8b_256(Xq, sx, Wq, sw, bias, M, N, K, Y, stream);
            }
            return QVGGT_ROWS(4, 4, 4, 1, 0, M);
        case GemmPlan::kSmall: return QVGGT_ROWS(2, 2, 3, 2, 0, M);
        case GemmPlan::kDeep: return QVGGT_ROWS(2, 2, 8, 1, 0, M);
        case GemmPlan::kBigThenDeep: break;
    }
    if constexpr (!ASYM) {
        if (acc_debug == nullptr) return launch_gemm_tail<CB, BLK>(Xq, sx, Wq, sw, bias, M, plan.rows_main, N, K, Y, stream);
    }
    const hipError_t e = QVGGT_ROWS(4, 4, 4, 1, 0, plan.rows_main);
    if (e != hipSuccess) return e;
    return QVGGT_ROWS(2, 2, 8, 1, plan.rows_main, M - plan.rows_main);
#undef QVGGT_ROWS
}

hipError_t run_w4a4_gemm(const uint8_t *Xq, const float *sx, const uint8_t *Wq, const float *sw,
                         const void *bias, int M, int N, int K, void *Y, int32_t *acc_debug, hipStream_t stream)
{
    if (M <= 0) return hipSuccess;
    return gemm_by_plan<4>(Xq, sx, Wq, sw, bias, M, N, K, Y, acc_debug, stream);
}

// Packed 4-bit codes with affine activations: Xq holds u - 8, xzero the zero points, wsum the weights' code sums per channel.
hipError_t run_w4a4_gemm_asym(const uint8_t *Xq, const float *sx, const float *xzero, const uint8_t *Wq, const float *sw,
                              const float *wsum, const void *bias, int M, int N, int K, void *Y, hipStream_t stream)
{
    if (M <= 0) return hipSuccess;
    return gemm_by_plan<4, true>(Xq, sx, Wq, sw, bias, M, N, K, Y, nullptr, stream, xzero, wsum);
}

// The same kernel on int8 codes (8- and 6-bit settings): rows of K bytes, no expansion, two K-steps per K-tile.
hipError_t run_i8_gemm(const int8_t *Xq, const float *sx, const int8_t *Wq, const float *sw, const void *bias, int M, int N,
                       int K, void *Y, int32_t *acc_debug, hipStream_t stream)
{
    if (M <= 0) return hipSuccess;
    const uint8_t *xq = reinterpret_cast<const uint8_t *>(Xq), *wq = reinterpret_cast<const uint8_t *>(Wq);
    return gemm_by_plan<8>(xq, sx, wq, sw, bias, M, N, K, Y, acc_debug, stream);
}

// int8 codes in 128-row blocks (see the kernel): whole tile rows go to either launch, so row offsets stay whole blocks
hipError_t run_i8b_gemm(const int8_t *Xb, const float *sx, const int8_t *Wb, const float *sw, const void *bias, int M, int N,
                        int K, void *Y, int32_t *acc_debug, hipStream_t stream)
{
    if (M <= 0) return hipSuccess;
    const uint8_t *xq = reinterpret_cast<const uint8_t *>(Xb), *wq = reinterpret_cast<const uint8_t *>(Wb);
    if (acc_debug == nullptr && i8b_resident(M, N, K))
        return run_i8b_resident({xq, sx, wq, sw, static_cast<const uint16_t *>(bias), M, N, K, static_cast<uint16_t *>(Y), nullptr, nullptr}, stream);
    return gemm_by_plan<8, false, true>(xq, sx, wq, sw, bias, M, N, K, Y, acc_debug, stream);
}

}  // namespace qvggt
