// One (output kind, outer mode) slice of the instantiations of the product kernel for small outputs; compiled once per slice
// with -DTJ_GEMM_OUT=0|1|2 -DTJ_GEMM_OUTER=0|1 -DTJ_GEMM_ARGS=GemmArgs|GemmGroup.
#include "gemm_kw_kernel.h"

#define TJ_CAT2(a, b, c, d) a##b##c##d
#define TJ_CAT(a, b, c, d) TJ_CAT2(a, b, c, d)

namespace tj {

hipError_t TJ_CAT(launch_gemm_kw_out, TJ_GEMM_OUT, _outer, TJ_GEMM_OUTER)(int tile, const TJ_GEMM_ARGS &g, dim3 grid, hipStream_t st)
{
    return launch_kw_tile<TJ_GEMM_OUT, TJ_GEMM_OUTER>(tile, g, grid, st);
}

}  // namespace tj
