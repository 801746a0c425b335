// The large-tile bf16 GEMM (gemm_large.h) with tiles of 256 x 256.
#include "gemm_large.h"

namespace mk {

bool launch_bgemm_large(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) { return launch_large<8>(p, st, t0, t1); }

int gemm_large_tiles(int M, int N) { return ((M + 255) / 256) * ((N + 255) / 256); }

}  // namespace mk
