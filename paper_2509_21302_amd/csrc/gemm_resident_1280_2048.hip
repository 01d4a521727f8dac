// The products with resident weights (gemm_resident.h) of K = 1280 and 2048.
#include "gemm_resident.h"

namespace qvggt {

template hipError_t launch_resident<E2m3Codes, 20, 1, false>(const ResidentProblem &, hipStream_t);
template hipError_t launch_resident<E2m3Codes, 16, 2, false>(const ResidentProblem &, hipStream_t);
static const LdsKernel resident_lds_kernel_list[] = {QVGGT_RESIDENT(E2m3Codes, 20, 1, false), QVGGT_RESIDENT(E2m3Codes, 16, 2, false)};
static const LdsKernels resident_lds_kernels(resident_lds_kernel_list);

}  // namespace qvggt
