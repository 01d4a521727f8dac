// The products with resident weights (gemm_resident.h): K = 512, 768, 1024 and int8 codes, and the way to the other sizes.
#include "gemm_resident.h"

namespace qvggt {

static const LdsKernel resident_lds_kernel_list[] = {
    QVGGT_RESIDENT(E2m3Codes, 8, 1, false), QVGGT_RESIDENT(E2m3Codes, 12, 1, false), QVGGT_RESIDENT(E2m3Codes, 16, 1, false), QVGGT_RESIDENT(Int8Codes, 16, 2, false)};
static const LdsKernels resident_lds_kernels(resident_lds_kernel_list);

// elsewhere: gemm_resident_1024_wide.hip, gemm_resident_1280_2048.hip, gemm_resident_1536_1792.hip, gemm_resident_affine.hip
extern template hipError_t launch_resident_tiles<E2m3Codes, 16, 1, 8, false>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 20, 1, false>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 16, 2, false>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 12, 2, false>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 14, 2, false>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 16, 1, true>(const ResidentProblem &, hipStream_t);
extern template hipError_t launch_resident<E2m3Codes, 16, 2, true>(const ResidentProblem &, hipStream_t);

// E2M3 blocks: the sizes of K are those of e2m3_resident_k; SHIFTED codes come with K = 1024 and 2048 only.
template <bool SHIFTED>
hipError_t run_e2m3_resident(const ResidentProblem &p, hipStream_t stream)
{
    switch (p.K) {
        case 1024:
            if constexpr (!SHIFTED) {
                if (resident_wide(p.M, p.N)) return launch_resident_tiles<E2m3Codes, 16, 1, 8, false>(p, stream);
            }
            return launch_resident<E2m3Codes, 16, 1, SHIFTED>(p, stream);
        case 2048: return launch_resident<E2m3Codes, 16, 2, SHIFTED>(p, stream);
    }
    if constexpr (!SHIFTED) {
        switch (p.K) {
            case 512: return launch_resident<E2m3Codes, 8, 1, false>(p, stream);
            case 768: return launch_resident<E2m3Codes, 12, 1, false>(p, stream);
            case 1280: return launch_resident<E2m3Codes, 20, 1, false>(p, stream);
            case 1536: return launch_resident<E2m3Codes, 12, 2, false>(p, stream);
            case 1792: return launch_resident<E2m3Codes, 14, 2, false>(p, stream);
        }
    }
    return hipErrorInvalidValue;
}
template hipError_t run_e2m3_resident<false>(const ResidentProblem &, hipStream_t);
template hipError_t run_e2m3_resident<true>(const ResidentProblem &, hipStream_t);

// int8 blocks, K = 1024
hipError_t run_i8b_resident(const ResidentProblem &p, hipStream_t stream)
{
    if (p.K != 1024) return hipErrorInvalidValue;
    hipError_t e = prepare_device();
    if (e != hipSuccess) return e;
    return launch_resident<Int8Codes, 16, 2, false>(p, stream);
}

}  // namespace qvggt
