// The large-tile bf16 GEMM (gemm_large.h) with tiles of 128 x 256.
#include "gemm_large.h"

namespace mk {

bool launch_bgemm_large128(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) { return launch_large<4>(p, st, t0, t1); }

}  // namespace mk
