// Shared between the translation units of the NT GEMM: kernel arguments, the per-instantiation launch entry points
// and the bf16 rounding both the product kernel and the split-K reduction use.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_fmt.h"

namespace tj {

constexpr int kGemmThreads = 256;
constexpr int kNumCU = 256;

// Where an operand's bytes are: row-major, or blocked along K as the backward quantizers write for the products (GemmOperand).  Strides of the
// codes by row and 64-k chunk, of the scale bytes by row and 256 k (four bytes per chunk inside), of the outer scales (floats) by row
// and 128 k.
struct OperandStrides {
    int64_t row, srow, grow, chunk, s256, g128;
};
__device__ __forceinline__ OperandStrides strides_of(bool blocked, int64_t rows, int64_t K)
{
    if (blocked) return OperandStrides{32, 16, 1, rows * 32, rows * 16, rows};
    return OperandStrides{K / 2, K / 16, K >> 7, 32, 16, 1};
}

struct GemmArgs {
    const uint8_t *a_codes, *a_scales;
    const uint8_t *b_codes, *b_scales;
    const float *a_gscale, *b_gscale;   // one float (tensor mode) or one per row and 128 k (block mode)
    void *out;          // bf16 / f32 [M x N], or f32 partials [split][M x N]
    int64_t M, N, K;
    int chunks_per_split;   // 64-wide K chunks per split
    int blocked;            // the operands are blocked along K (gemm_nt_kernel, all products of a group alike; the other kernel reads row-major ones)
    int tiles_m, tiles_n;
    int out_f32;
    int outer;              // 0 one outer scale per operand, 1 one per row and 128 k
};

// Up to three independent products of one launch: product i has the workgroups from first[i] on (in the grid's x dimension;
// INT_MAX where there is none).
constexpr int kMaxGroup = 3;
struct GemmGroup {
    int first[kMaxGroup];
    GemmArgs g[kMaxGroup];
};

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    const uint32_t b = f2u(f);
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

// One translation unit per (output kind, scale-fetch variant, outer mode) instantiates the product kernel for every
// tile shape: out 0 bf16, 1 f32, 2 raw f32 split-K partial; ps = paired scale fetch (K a multiple of 256); outer = 1:
// one FP32 outer scale per row and 128 k.  tile: 0 256x256 (outer 0 only), 1 256x128, 2 128x256, 3 128x128,
// 4 128x192 (ps only), 5 64x64 (outer 0: one product in one piece, short reductions), 6 64x128 (ps only).
// Each for one product and, but for the partials, for a group.
#define TJ_DECL_GEMM_INST(ps, out, outer) \
    hipError_t launch_gemm_inst_ps##ps##_out##out##_outer##outer(int tile, const GemmArgs &g, dim3 grid, hipStream_t st); \
    hipError_t launch_gemm_inst_ps##ps##_out##out##_outer##outer(int tile, const GemmGroup &g, dim3 grid, hipStream_t st);
TJ_DECL_GEMM_INST(0, 0, 0) TJ_DECL_GEMM_INST(0, 1, 0) TJ_DECL_GEMM_INST(0, 2, 0)
TJ_DECL_GEMM_INST(1, 0, 0) TJ_DECL_GEMM_INST(1, 1, 0) TJ_DECL_GEMM_INST(1, 2, 0)
TJ_DECL_GEMM_INST(0, 0, 1) TJ_DECL_GEMM_INST(0, 1, 1) TJ_DECL_GEMM_INST(0, 2, 1)
TJ_DECL_GEMM_INST(1, 0, 1) TJ_DECL_GEMM_INST(1, 1, 1) TJ_DECL_GEMM_INST(1, 2, 1)
#undef TJ_DECL_GEMM_INST
// The kernel whose waves split the reduction, for any K >= 256 (outer 1: 768): tile 5 64x64, 6 64x128, 7 128x128 (outer 0 only, no
// partials).
#define TJ_DECL_GEMM_KW(out, outer) \
    hipError_t launch_gemm_kw_out##out##_outer##outer(int tile, const GemmArgs &g, dim3 grid, hipStream_t st); \
    hipError_t launch_gemm_kw_out##out##_outer##outer(int tile, const GemmGroup &g, dim3 grid, hipStream_t st);
TJ_DECL_GEMM_KW(0, 0) TJ_DECL_GEMM_KW(1, 0) TJ_DECL_GEMM_KW(2, 0)
TJ_DECL_GEMM_KW(0, 1) TJ_DECL_GEMM_KW(1, 1) TJ_DECL_GEMM_KW(2, 1)
#undef TJ_DECL_GEMM_KW

}  // namespace tj
