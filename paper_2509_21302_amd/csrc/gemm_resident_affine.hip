// The products with resident weights (gemm_resident.h) of affine codes.
#include "gemm_resident.h"

namespace qvggt {

template hipError_t launch_resident<E2m3Codes, 16, 1, true>(const ResidentProblem &, hipStream_t);
template hipError_t launch_resident<E2m3Codes, 16, 2, true>(const ResidentProblem &, hipStream_t);
static const LdsKernel resident_lds_kernel_list[] = {QVGGT_RESIDENT(E2m3Codes, 16, 1, true), QVGGT_RESIDENT(E2m3Codes, 16, 2, true)};
static const LdsKernels resident_lds_kernels(resident_lds_kernel_list);

}  // namespace qvggt
