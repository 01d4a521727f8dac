// The products with the weights resident in registers (gemm_resident.h), for the problems that the rules of gemm_plan.h give them.
#pragma once
#include "qvggt_common.h"

namespace qvggt {

struct ResidentProblem {
    const uint8_t *Xq;      // blocks of 128 rows of either format, whole blocks
    const float *sx;
    const uint8_t *Wq;
    const float *sw;
    const uint16_t *bias;
    int M, N, K;
    uint16_t *Y;
    const float *xzero, *wsum;      // with SHIFTED codes
};

template <bool SHIFTED>
hipError_t run_e2m3_resident(const ResidentProblem &p, hipStream_t stream);
hipError_t run_i8b_resident(const ResidentProblem &p, hipStream_t stream);

}  // namespace qvggt
