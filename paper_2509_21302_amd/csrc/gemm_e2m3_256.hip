// The E2M3 product in tiles of 256 tokens x 256 channels (gemm_tiles256.h; gemm_e2m3.hip has the operand format, the other shapes and the choice among them): many
// tokens of long K.  A K-step is two units of the format, a ring of three stages.
//
// What bounds it, 137400 x 4096 -> 1024, 308 us (32x32x64: 320): the way from memory into LDS.  A pair of units takes 1615 cycles at 1.94 GHz, 64 MFMAs of 16 among
// them; waiting at the barrier is 130, the rest is transfer instructions that the full memory pipeline does not take.  With the tokens of all tiles the same
// ones, in the L2: 253 us; without transfers 222, without transfers and LDS reads 190; without the stores 265; all codes zero 298, so that it is not the
// board's power.  Tried and not better: the tokens' lines brought into the L2 one to six pairs ahead (each block a quarter of them; 305), K walked from another place
// in every tile, transfers issued faster (312), waits that leave the epilogue's stores in flight.  192 tokens in this form: 30.8 us at
// 10992 x 4096 -> 1024, 28.7 in the kernel of gemm_e2m3.hip.
#include "gemm_tiles256.h"

#include <algorithm>

namespace qvggt {

template <bool DEBUG, bool SHIFTED, bool STREAM_Y>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void e2m3_256_kernel(
    const uint8_t *__restrict__ Xf, const float *__restrict__ sx, const uint8_t *__restrict__ Wf,
    const float *__restrict__ sw, const uint16_t *__restrict__ bias, int M, int N, int K,
    uint16_t *__restrict__ Y, int32_t *__restrict__ acc_debug, int tiles_m, int tiles_n,
    const float *__restrict__ xzero, const float *__restrict__ wsum)
{
    tiles256<E2m3Tiles, DEBUG, SHIFTED, STREAM_Y>(Xf, sx, Wf, sw, bias, M, N, K, Y, acc_debug, tiles_m, tiles_n, xzero, wsum);
}

// every instantiation launched below, with the dynamic LDS it needs
#define QVGGT_256_KERNEL(DEBUG, SHIFTED, STREAM_Y) {reinterpret_cast<const void *>(e2m3_256_kernel<DEBUG, SHIFTED, STREAM_Y>), Cfg256<E2m3Tiles, SHIFTED>::LDS_BYTES}
static const LdsKernel e2m3_256_lds_kernel_list[] = {QVGGT_256_KERNEL(false, false, true), QVGGT_256_KERNEL(false, false, false), QVGGT_256_KERNEL(true, false, true),
                                                     QVGGT_256_KERNEL(false, true, true), QVGGT_256_KERNEL(false, true, false)};
#undef QVGGT_256_KERNEL
static const LdsKernels e2m3_256_lds_kernels(e2m3_256_lds_kernel_list);

template <bool SHIFTED>
hipError_t run_e2m3_256(const E2m3Problem &p, hipStream_t stream)
{
    using C = Cfg256<E2m3Tiles, SHIFTED>;
    if (p.K < TILES256_LEAST_K) return hipErrorInvalidValue;
    const int tiles_m = (p.M + C::BM - 1) / C::BM, tiles_n = (p.N + C::BN - 1) / C::BN;
    auto kern = e2m3_streams_y(p.M, p.N) ? e2m3_256_kernel<false, SHIFTED, true> : e2m3_256_kernel<false, SHIFTED, false>;
    if constexpr (!SHIFTED) {
        if (p.acc_debug != nullptr) kern = e2m3_256_kernel<true, false, true>;
    }
    const int grid = std::min(256, (tiles_m * tiles_n + 7) / 8 * 8);
    kern<<<grid, C::THREADS, C::LDS_BYTES, stream>>>(p.Xf, p.sx, p.Wf, p.sw, p.bias, p.M, p.N, p.K, p.Y, p.acc_debug, tiles_m, tiles_n, p.xzero, p.wsum);
    return hipGetLastError();
}
template hipError_t run_e2m3_256<false>(const E2m3Problem &, hipStream_t);
template hipError_t run_e2m3_256<true>(const E2m3Problem &, hipStream_t);

}  // namespace qvggt
