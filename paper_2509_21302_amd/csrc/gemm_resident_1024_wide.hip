// The products with resident weights (gemm_resident.h): K = 1024 with 128 channels a wave.
#include "gemm_resident.h"

namespace qvggt {

static const LdsKernel resident_lds_kernel_list[] = {QVGGT_RESIDENT_TILES(E2m3Codes, 16, 1, 8, false, true)};
static const LdsKernels resident_lds_kernels(resident_lds_kernel_list);

template hipError_t launch_resident_tiles<E2m3Codes, 16, 1, 8, false>(const ResidentProblem &, hipStream_t);

}  // namespace qvggt
