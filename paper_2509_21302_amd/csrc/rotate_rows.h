// One row per wavefront: how a row of K values (K a power of two, 128 .. 8192) is spread over the 64 lanes, loaded, and taken
// through the unnormalised Walsh-Hadamard transform.  Shared by the generic kernel 1 and the calibration-side rotation.
//
// A row of K values lives in K/64 registers per lane; element e = c*(64*V) + lane*V + i sits in register c*V + i, where
// V = min(8, K/64) is the run a lane loads contiguously (16 bytes of bf16 when V = 8, so a wave reads 1 KiB per load
// instruction).  The transform is one butterfly per index bit (the Hadamard matrix is a Kronecker power of H_2, paper Sec. 3.2):
// bits inside i and c are register-to-register, the six lane bits go through cross-lane exchanges.
#pragma once
#include "qvggt_common.h"

namespace qvggt {

template <int K>
struct RowMap {
    static constexpr int V = (K >= 512) ? 8 : K / 64;   // contiguous elements per lane per chunk
    static constexpr int C = K / (64 * V);              // chunks
    static constexpr int R = V * C;                     // registers per lane
};

template <int K, bool F32>
__device__ inline void load_row(const void *X, size_t row, int lane, float (&x)[RowMap<K>::R])
{
    constexpr int V = RowMap<K>::V, C = RowMap<K>::C;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const size_t e0 = row * (size_t)K + (size_t)c * 64 * V + (size_t)lane * V;
        if constexpr (F32) {
            const float *p = reinterpret_cast<const float *>(X) + e0;
            if constexpr (V >= 4) {
#pragma unroll
                for (int q = 0; q < V / 4; ++q) {
                    float4 v = *reinterpret_cast<const float4 *>(p + 4 * q);
                    x[c * V + 4 * q + 0] = v.x; x[c * V + 4 * q + 1] = v.y;
                    x[c * V + 4 * q + 2] = v.z; x[c * V + 4 * q + 3] = v.w;
                }
            } else {
                float2 v = *reinterpret_cast<const float2 *>(p);
                x[c * V] = v.x; x[c * V + 1] = v.y;
            }
        } else {
            const uint16_t *p = reinterpret_cast<const uint16_t *>(X) + e0;
            uint32_t w[V / 2];
            if constexpr (V == 8) {
                uint4 v = *reinterpret_cast<const uint4 *>(p);
                w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
            } else if constexpr (V == 4) {
                uint2 v = *reinterpret_cast<const uint2 *>(p);
                w[0] = v.x; w[1] = v.y;
            } else {
                w[0] = *reinterpret_cast<const uint32_t *>(p);
            }
#pragma unroll
            for (int q = 0; q < V / 2; ++q) {
                x[c * V + 2 * q] = __uint_as_float(w[q] << 16);
                x[c * V + 2 * q + 1] = __uint_as_float(w[q] & 0xFFFF0000u);
            }
        }
    }
}

// In-place unnormalised Walsh-Hadamard transform of a row spread over one wavefront.
template <int K>
__device__ inline void fwht_row(float (&x)[RowMap<K>::R], int lane)
{
    constexpr int V = RowMap<K>::V, R = RowMap<K>::R;
    // index bits inside the lane's contiguous run
#pragma unroll
    for (int h = 1; h < V; h <<= 1)
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((r & h) == 0) { float a = x[r], b = x[r + h]; x[r] = a + b; x[r + h] = a - b; }
    lane_butterflies(x, lane);
    // chunk bits
#pragma unroll
    for (int h = V; h < R; h <<= 1)
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((r & h) == 0) { float a = x[r], b = x[r + h]; x[r] = a + b; x[r + h] = a - b; }
}

// ---- E2M3 output of the row kernels (format: gemm_e2m3.hip).  A row's codes go to LDS as bytes at their positions; a group of consecutive rows
// leaves together.  Groups are four rows, so that memory sees runs of 192 bytes per unit: single rows' 48-byte pieces of lines, written by blocks
// of different XCDs, are what it takes worst.  (Where a block's four waves share a row, a group is one row while there are few rows: four rows one
// after the other on a quarter of the blocks take longer, 732 x 6144 39 against 35 us with its GEMM.)  Writing this form costs a kernel that is
// bound by the vector ALU 10 to 15 % over packed codes.
constexpr int kE2m3Group = 4;
constexpr int kFewSharedRows = 4096;         // two rounds of 2048 blocks of one row
template <int K>
struct E2m3Stage {
    static constexpr int PITCH = K + 64;                // the rows start in different quarters of the banks
    static constexpr int BYTES = kE2m3Group * PITCH;
};

// the low bytes of four words as one
__device__ inline uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0C0C0400u), __builtin_amdgcn_perm(b, a, 0x0C0C0400u), 0x05040100u);
}

// 32 codes (bytes, two's complement, in [-7, 7], 16-byte aligned) as the 24 bytes of an E2M3 blob
typedef unsigned int e2m3_v6u __attribute__((ext_vector_type(6)));
__device__ inline e2m3_v6u e2m3_blob(const uint8_t *p)
{
    typedef float v16f __attribute__((ext_vector_type(16)));
    const uint4 lo = *reinterpret_cast<const uint4 *>(p), hi = *reinterpret_cast<const uint4 *>(p + 16);
    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    v16f ev, od;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const uint32_t v = w[d] ^ 0x80808080u;
        ev[2 * d] = (float)(v & 0xFFu) - 128.0f;
        od[2 * d] = (float)((v >> 8) & 0xFFu) - 128.0f;
        ev[2 * d + 1] = (float)((v >> 16) & 0xFFu) - 128.0f;
        od[2 * d + 1] = (float)(v >> 24) - 128.0f;
    }
    e2m3_v6u blob;           // early clobber: the conversion writes results while it still reads its sources (see the matrix-core kernel)
    asm volatile("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, 1.0" : "=&v"(blob) : "v"(ev), "v"(od));
    return blob;
}

// 32 codes (bytes, two's complement) as the 16 bytes of packed nibbles
__device__ inline uint4 packed_codes(const uint8_t *p)
{
    const uint4 lo = *reinterpret_cast<const uint4 *>(p), hi = *reinterpret_cast<const uint4 *>(p + 16);
    auto nibbles = [](uint32_t a, uint32_t b) {
        const uint32_t x = (a & 0x0F0F0F0Fu) | (a & 0x0F0F0F0Fu) >> 4, y = (b & 0x0F0F0F0Fu) | (b & 0x0F0F0F0Fu) >> 4;      // pairs in bytes 0 and 2
        return __builtin_amdgcn_perm(y, x, 0x06040200u);
    };
    return make_uint4(nibbles(lo.x, lo.y), nibbles(lo.z, lo.w), nibbles(hi.x, hi.y), nibbles(hi.z, hi.w));
}

// 256 threads write the staged codes of rows row0 .. row0 + group - 1 (a group of four or one), as far as they exist; BOTH: to packed rows as well.
// Between two barriers.
template <int K, bool BOTH>
__device__ inline void flush_e2m3(const uint8_t *stage, int row0, int group, int rows, uint8_t *out, uint8_t *rows_out)
{
    uint8_t *block = out + (size_t)(row0 / 128) * (K / 64) * 6144 + (size_t)(row0 % 128) * 48;
    for (int t = threadIdx.x; t < K / 32 * group; t += 256) {          // 32 codes each: unit, row, half
        const int h = t & 1, r = (t >> 1) & (group - 1), unit = (t >> 1) / group;
        if (row0 + r >= rows) continue;
        const uint8_t *codes = stage + r * E2m3Stage<K>::PITCH + 64 * unit + 32 * h;
        if constexpr (BOTH) *reinterpret_cast<uint4 *>(rows_out + (size_t)(row0 + r) * (K / 2) + 32 * unit + 16 * h) = packed_codes(codes);
        const e2m3_v6u blob = e2m3_blob(codes);
        uint8_t *u = block + (size_t)unit * 6144 + r * 48;
        *reinterpret_cast<uint4 *>(u + h * 16) = make_uint4(blob[0], blob[1], blob[2], blob[3]);
        *reinterpret_cast<uint2 *>(u + 32 + h * 8) = make_uint2(blob[4], blob[5]);
    }
}

}  // namespace qvggt
