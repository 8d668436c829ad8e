// Host side of the NT GEMM on two packed NVFP4 operands (tile / split planner, launcher) and the split-K reduction.
// The product kernel itself lives in gemm_kernel.h and is instantiated slice by slice in gemm_inst.hip.
#include <climits>
#include <utility>

#include "../../include/tjnvfp4.h"
#include "gemm_args.h"
#include "internal.h"

namespace tj {

namespace {

constexpr int kThreads = kGemmThreads;
constexpr int kNC = 2;

// K = 0: the product is all zeros (no operand, and no outer scale, is looked at)
__global__ __launch_bounds__(kThreads) void zero_out_kernel(uint16_t *out, int64_t n16)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n16; i += stride) out[i] = 0;
}

// partials are read exactly once: streaming load
__device__ __forceinline__ float4 ld4(const float *p)
{
    const float4_t v = __builtin_nontemporal_load(reinterpret_cast<const float4_t *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

// sum the split-K partials in split order, scale, convert
__global__ __launch_bounds__(kThreads) void splitk_reduce_kernel(const float *__restrict__ part, int split,
                                                                 int64_t mn, const float *a_gscale,
                                                                 const float *b_gscale, int outer, void *out, int out_f32)
{
    // block mode: the partial sums already carry the outer scales
    const float alpha = outer ? 256.0f : a_gscale[0] * b_gscale[0] * 256.0f;
    const int64_t i4 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (i4 >= mn) return;
    if ((mn & 3) == 0) {
        float4 s = ld4(part + i4);
        for (int z = 1; z < split; ++z) {
            const float4 t = ld4(part + (int64_t)z * mn + i4);
            s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        s.x *= alpha; s.y *= alpha; s.z *= alpha; s.w *= alpha;
        if (out_f32) {
            *reinterpret_cast<float4 *>(reinterpret_cast<float *>(out) + i4) = s;
        } else {
            uint2 p;
            p.x = f32_to_bf16_bits(s.x) | (f32_to_bf16_bits(s.y) << 16);
            p.y = f32_to_bf16_bits(s.z) | (f32_to_bf16_bits(s.w) << 16);
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + i4) = p;
        }
    } else {
        for (int64_t i = i4; i < mn && i < i4 + 4; ++i) {
            float s = part[i];
            for (int z = 1; z < split; ++z) s += part[(int64_t)z * mn + i];
            s *= alpha;
            if (out_f32) reinterpret_cast<float *>(out)[i] = s;
            else reinterpret_cast<uint16_t *>(out)[i] = (uint16_t)f32_to_bf16_bits(s);
        }
    }
}

// ---- host side: tile shape and split choice ---------------------------------------------------

// Tile shapes and a small cost model (microseconds, from timings of this kernel on MI355X) that picks
// the tile and the number of K splits for a problem.
struct TileCfg { int tm, tn; double t_stage; double t_fixed; int occupancy; };
// t_stage: one 128-k pipeline stage of one workgroup with the CU to itself; t_fixed: prologue + epilogue
// the 128 x 192 tile exists for the paired scale fetch only (K a multiple of 256)
const TileCfg kTiles[] = {{4, 4, 3.2, 6.0, 1}, {4, 2, 2.0, 5.0, 1}, {2, 4, 2.0, 5.0, 1}, {2, 2, 1.5, 5.0, 3}, {2, 3, 1.4, 5.0, 2},
                          {1, 1, 0.6, 3.2, 3}, {1, 2, 0.9, 3.2, 2}, {2, 2, 1.5, 5.0, 1}};
constexpr int kNumTiles = 8;
// Costs fitted to sustained runs of the tiles on whole layers' products (64 x 64 to 256 x 256 tiles; 1000 to 16384 rows, K =
// 512 .. 16384), here with t_fixed shared between the workgroups of a CU like the stages: [0] per-tensor scales, [1]
// 1 x 128 outer blocks, whose rescale in every stage and second accumulator set change the tiles' order.  Examples: 1000 x
// 3072 x 1024 12.8 us with 128 x 128, 15.8 with 128 x 192; with outer blocks 8192 x 4096 x 4096 311 us with 128 x 128, 320 with 256 x 128,
// 385 with 128 x 192, and 2048 x 2048 x 2048 28.4 us with 128 x 128, 40.1 with 256 x 128.  They are used for outputs of at least 128 rows
// and columns, ragged ones included (360 random ragged shapes where the two sets differ: these are 1.17 times as fast
// with per-tensor scales and 1.13 with outer blocks; eight of them are 0.80 to 0.9), and from the reduction length on at which they become the
// better set: 512 with per-tensor scales (64 to 448: 0.85 times as fast as the costs above; 1384 x 2488 x 512: 9.6 us against
// 11.3), 256 with outer blocks (256 to 640, 160 shapes: 1.16 times as fast, 3027 x 896 x 256 8.1 us against 9.7; 128: 506 x 2496
// 7.1 against 5.6).  Slivers keep the costs above.
const TileCfg kTilesFit[2][kNumTiles] = {
    {{4, 4, 2.9, 7.2, 1}, {4, 2, 1.78, 4.0, 1}, {2, 4, 1.78, 4.0, 1}, {2, 2, 1.1, 4.0, 2}, {2, 3, 1.33, 5.2, 2}, {1, 1, 0.285, 3.9, 2}, {1, 2, 0.55, 5.3, 1}, {2, 2, 0.84, 7.3, 1}},
    {{4, 4, 0, 0, 1}, {4, 2, 2.48, 3.2, 1}, {2, 4, 2.57, 3.2, 1}, {2, 2, 1.52, 4.0, 2}, {2, 3, 2.0, 3.3, 1}, {1, 1, 0.41, 4.6, 1}, {1, 2, 0.78, 5.6, 1}, {2, 2, 0, 0, 1}}};
// Tiles 5, 6 and 7 above are costs of gemm_kw_kernel, for whole outputs (rows and columns in 64s).  Measured: 64 x 64 with one
// workgroup per CU 3.9 us + 0.29 per 128 k (1024 x 1024: K = 512 5.3 us, 1024 6.5, 2048 8.9), with two 5.5 + 0.5; 64 x 128 5.4 +
// 0.57 (2048 x 1024 x 1024 9.9); 128 x 128 7.3 + 0.6 to 0.8 (2048 x 2048 x 2048 19.7 us, 20.8 with gemm_nt_kernel's tile of that size;
// 2752 x 1088 x 4416 33.5, 41.5); with outer blocks 64 x 64 4.6 + 0.41 and 64 x 128 5.6 + 0.78.  Ragged outputs keep the costs that the
// 64 x 64 and 64 x 128 tiles have in gemm_nt_kernel: those are tested on ragged shapes, these are fitted to whole ones only, and waves_split_k then takes the kernel
// that is the faster one for the tile and split that they give.
const TileCfg kSmallRagged[2][2] = {{{1, 1, 0.6, 3.2, 3}, {1, 2, 0.85, 3.2, 2}}, {{1, 1, 0.81, 3.2, 3}, {1, 2, 1.2, 3.2, 2}}};

// Whether the 64 x 64 (5) and 64 x 128 (6) tiles run on gemm_kw_kernel, for a reduction of `chunks` 64s per split: below these its four
// waves have too little to share (device times of 700 random shapes, gemm_nt_kernel's over gemm_kw_kernel's: 64 x 64, 4 to 6 chunks
// 1.00, 7 1.10, 12 1.1 to 1.25, 30 1.4; 64 x 128, 8 chunks 0.96, 12 0.99, 16 1.06; with outer blocks 64 x 64, 10 chunks 0.99, 12 1.06, 14 1.2,
// 64 x 128, 12 chunks 0.95, 16 1.1).
// ragged_wgs: the workgroups of a ragged output, 0 for a whole one.  The kernel's rings and closing sums leave room for two workgroups on a
// CU with the 64 x 64 tile, for one with 64 x 128 and with outer blocks, where gemm_nt_kernel runs three.  A ragged output is planned with the
// latter's costs, so it may come with more workgroups than that; they are left to that kernel (gemm_kw_kernel would have 0.72 to 0.98 of
// its speed with outer blocks - 275 x 2895 x 3072 32.5 us against 26.1, 2162 x 513 x 1152 20.0 against 17.0 -, 0.91 to 0.97 with 64 x 128; from 30 chunks on
// it has 1.02), as are the shortest reductions (64 x 64 on more than 256 workgroups, 5 and 6 chunks 0.95, 7 1.08; 64 x 128 with outer
// blocks, see above): 160 random shapes that change kernel by it are 1.08 times as fast, 1.00 at worst.  Whole outputs are planned with this kernel's own
// costs, and keep it for the shortest reductions too, because the products of a backward call, which are all whole, share a
// launch only if they run the same kernel (320 x 960 -> 1536: the call's launches 19.8 us together, 25.2 one by one).
bool waves_split_k(int tile, int64_t chunks, int64_t ragged_wgs, int outer)
{
    if (tile == 7) return true;
    if (tile < 5) return false;
    const bool crowded = ragged_wgs > kNumCU;
    if (crowded && (tile == 6 || outer)) return chunks >= 30;
    return chunks >= (tile == 6 ? (outer && ragged_wgs > 0 ? 13 : 12) : outer ? 12 : crowded ? 7 : 4);
}

// kFitted: the fitted costs where they hold; kUnfitted: the costs above for every shape; kEarly: those without the small tiles
enum Costs { kFitted, kUnfitted, kEarly };
Plan rank_tiles(int64_t M, int64_t N, int64_t K, int outer, Costs costs)
{
    const bool early = costs == kEarly;
    const int64_t chunks = K / 64;
    Plan best{3, 1, (int)chunks, false, 0.0};
    if (M <= 0 || N <= 0 || chunks == 0) return best;      // nothing to tile (empty output or empty reduction)
    double best_t = 1e300;
    const bool fit = costs == kFitted && M >= 128 && N >= 128 && K >= (outer ? 256 : 512);
    const bool whole = M % 64 == 0 && N % 64 == 0;
    for (int t = 0; t < kNumTiles; ++t) {
        if (t == 4 && K % 256 != 0) continue;
        // The small tiles are for outputs that leave CUs idle with 128 x 128 workgroups: there the time is the chain of a
        // tile's stages, and a 64-row tile's stage is half as long (256 x 512 x 512: 9.6 us with 128 x 192, 5.6 with
        // 64 x 64; 2048 x 1024 x 1024: 14.6 us with 128 x 192, 10.4 with 64 x 128); longer chains than 16 stages are split
        // instead (768 x 768 x 3072: 15.5 against 20.0, 512 x 512 x 8192: 17.3 against 23.3, 1000 x 520 x 3072: 16.2 against 20.2).  A
        // filled chip pays for them with twice the expansions per product (8192 x 3072 x 768: 73 us with
        // 64 x 64, 42 with 128 x 192), and a sliver of an output with
        // rows that are mostly padding.  With 1 x 128 outer blocks the same holds (2048 x 1024 x 1024: 19.8 us with 128 x 192),
        // a little earlier where only the 64 x 64 tile exists.
        // Whole outputs with per-tensor scales may take any number of 64 x 64 tiles of gemm_kw_kernel in one piece (`many`): two on a CU
        // have nearly the rate of the 128 x 128 tile, with a quarter of its granularity.  Measured with r rounds of 512 of them
        // (us, and the best other plan): r = 0.96 1088 x 1856 x 14400 67 (84), 1.74 11392 x 320 x 7104 68 (98), 1.95 1728 x 2368 x 4224 42 (58),
        // 2.3 4416 x 1088 x 2752 37.5 (48.3), 2.4 5696 x 896 x 6016 71 (88); but 3.4 2688 x 2624 x 13632 214 (192).  All follow 5 us +
        // 1.3 per round + 0.54 per round and stage, a last round that is begun after the second counting 0.4 more than its share; a
        // plan of at most four rounds (the measured range) has to be 8 % better by that, because the other tiles' costs are that much too high for some long reductions (11136 x
        // 384 x 6656 63, 71 with 64 x 64).
        bool many = false;
        if (t == 5 || t == 6) {
            if (early) continue;
            const int64_t least = outer ? 256 : 128, tiles128 = ((M + 127) / 128) * ((N + 127) / 128);
            if (M < least || N < least) continue;
            if (tiles128 > (outer && K % 256 != 0 ? 3 * kNumCU / 8 : kNumCU / 2)) {
                if (t == 6 || outer || !fit || !whole) continue;
                many = true;
            }
        }
        if (t == 7 && (!fit || !whole || outer)) continue;
        if (t == 0 && outer) continue;                      // block mode keeps two accumulator sets: at most 2 x 4 tiles per wave
        const int64_t bm = 64 * kTiles[t].tm, bn = 64 * kTiles[t].tn;
        const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        for (int split = 1; split <= 16; ++split) {
            if (split > 1 && (chunks / split < 8 || t == 7 || many)) break;
            int64_t cps = (chunks + split - 1) / split;
            if (chunks % 4 == 0) cps = (cps + 3) / 4 * 4;                       // splits on 256-k boundaries
            else if (outer) cps = (cps + 1) / 2 * 2;                            // block mode: on 128-k boundaries
            if (split > 1 && (chunks + cps - 1) / cps != split) continue;      // same launch as a smaller split
            const int64_t wgs = tiles * split;
            const bool runs_kw = waves_split_k(t, cps, whole ? 0 : wgs, outer), kw = fit && whole && runs_kw;   // kw: and has its costs
            if (t == 6 && K % 256 != 0 && !kw) continue;             // the other kernel has no such instantiation
            if (t >= 5 && !kw && cps > 16 * kNC) continue;                                          // small tiles: at most 16 stages
            const double stages = (double)((cps + kNC - 1) / kNC);
            // workgroups sharing a CU slow each other down (128 x 128 tiles: up to three per CU)
            const int64_t per_cu = (wgs + kNumCU - 1) / kNumCU;
            const TileCfg &cfg = !fit ? kTiles[t] : t >= 5 && !kw ? kSmallRagged[outer][t - 5] : kTilesFit[outer][t];
            // A third 128 x 128 workgroup with outer blocks still runs beside the other two when it makes the launch a single round
            // (513 to 768 tiles in one piece: 16640 x 640 x 256 17.8 us, 21.8 with 256 x 128; 76 shapes 1.07 times as fast, 0.98 at
            // worst); above K = 3072 split plans are the better ones (1600 x 5888 x 8320: 279 us with 256 x 128 in three, 311), and
            // counted on in every round it costs 10 % on larger outputs (9674 x 7936 x 4480: 1079 against 968 us).
            const bool third = fit && outer && t == 3 && split == 1 && per_cu == 3 && K <= 3072;
            const int64_t conc = third ? 3 : per_cu < cfg.occupancy ? per_cu : cfg.occupancy;
            // (unfitted, 128 x 192: 1.9 with a split, where 1.75 made slivers take twice the splits - 35 x 7058 x 5632 with outer
            // blocks 37.5 against 28.2 us, 106 x 8529 x 13056 63.6 against 47.0; 1.75 without one, where 1.9 gave short reductions
            // 256 x 256 tiles - 12864 x 4288 x 256 55.7 us against 46.4)
            const double slow = conc == 1 ? 1.0
                                : fit     ? (conc > 2 ? 1.95 : t >= 5 && !kw ? 1.4 : outer ? (K < 512 || split > 1 ? 1.7 : 1.52) : 1.58)
                                : conc == 2 ? (t == 4 && split > 1 && !early ? 1.9 : 1.75) : 2.35;
            // (outer blocks: 1.52 is the 128 x 128 tile's since it keeps both accumulator sets in ordinary registers; split plans keep
            // the 1.7 from before, so that no product comes to need a workspace by it.  125 random products that take that tile instead of a larger one
            // for the 1.52: 1.07 times as fast, up to 1.32 where the larger tile's second round is short, 0.97 to 1.00 at 290 to 490 tiles
            // of long reductions - 3072 x 2432 x 20224 360 -> 372 us)
            const int64_t waves = (wgs + kNumCU * conc - 1) / (kNumCU * conc);
            // 128 x 128 with split waves: a stage takes longer the more CUs draw on the L2 caches (144 workgroups 0.64 us, 198 0.76, 256 0.8)
            const double t_stage = t == 7 ? 0.55 + 0.29 * (wgs < kNumCU ? (double)wgs / kNumCU : 1.0) : cfg.t_stage;
            // unfitted block mode: the per-block rescale of the accumulators makes a stage about a third longer
            double time = fit ? (double)waves * (stages * t_stage + cfg.t_fixed) * slow
                              : (double)waves * (stages * cfg.t_stage * (outer ? 1.35 : 1.0) * slow + cfg.t_fixed);
            if (many) {
                const double r = (double)wgs / (2 * kNumCU), up = (double)((wgs + 2 * kNumCU - 1) / (2 * kNumCU));
                const double rounds = r > 2.0 && r + 0.4 < up ? r + 0.4 : up;
                time = r > 4.0 ? 1e300 : rounds * (stages * 0.54 + 1.3) + 5.0;
            }
            // partials out and back in (768 x 768 x 8192: 64 x 64 tiles of gemm_kw_kernel in three 22.1 us, in one piece 22.6)
            if (split > 1) time += (kw && !outer ? 3.2 : 4.0) + (double)(split + 1) * (double)(M * N) * 4.0 / 3.5e6;
            const double rank = many ? 1.08 * time : time;
            if (rank < best_t) { best_t = rank; best = Plan{t, split, (int)cps, runs_kw, time}; }
        }
    }
    return best;
}

size_t split_bytes(const Plan &p, int64_t M, int64_t N) { return p.split > 1 ? (size_t)p.split * (size_t)M * (size_t)N * sizeof(float) : 0; }

Plan make_plan(int64_t M, int64_t N, int64_t K, int outer)
{
    const Plan p = rank_tiles(M, N, K, outer, kFitted);
    if (split_bytes(p, M, N) <= (size_t)NVFP4_STATIC_SCRATCH_BYTES) return p;
    // A better split must not put a product out of reach of the entry point with a fixed scratch array: where one of the
    // earlier sets of costs gives a plan that fits it, that plan stays (0.7 % of the shapes with 64 to 20000 rows and columns).
    for (const Costs c : {kUnfitted, kEarly}) {
        const Plan q = rank_tiles(M, N, K, outer, c);
        if (split_bytes(q, M, N) <= (size_t)NVFP4_STATIC_SCRATCH_BYTES) return q;
    }
    return p;
}

GemmArgs args_of(const GemmOperand &A, const GemmOperand &B, int64_t K, void *out, int out_f32, int tile, int chunks_per_split)
{
    GemmArgs g;
    g.a_codes = A.codes; g.a_scales = A.scales; g.a_gscale = A.gscale;
    g.b_codes = B.codes; g.b_scales = B.scales; g.b_gscale = B.gscale;
    g.M = A.rows; g.N = B.rows; g.K = K;
    const int bm = 64 * kTiles[tile].tm, bn = 64 * kTiles[tile].tn;
    g.tiles_m = (int)((g.M + bm - 1) / bm);
    g.tiles_n = (int)((g.N + bn - 1) / bn);
    g.chunks_per_split = chunks_per_split;
    g.out_f32 = out_f32;
    g.outer = A.outer;
    g.blocked = A.blocked;
    g.out = out;
    return g;
}

// kind: 0 bf16, 1 f32, 2 split partials; ps: K a multiple of 256 with splits on 256-boundaries, scale bytes fetched 16 per row;
// kw: the kernel whose waves split the reduction
hipError_t launch_tiles(int tile, int outer, bool ps, int kind, bool kw, const GemmArgs &g, dim3 grid, hipStream_t st)
{
    typedef hipError_t (*InstFn)(int, const GemmArgs &, dim3, hipStream_t);
    static const InstFn inst[2][2][3] = {
        {{launch_gemm_inst_ps0_out0_outer0, launch_gemm_inst_ps0_out1_outer0, launch_gemm_inst_ps0_out2_outer0},
         {launch_gemm_inst_ps1_out0_outer0, launch_gemm_inst_ps1_out1_outer0, launch_gemm_inst_ps1_out2_outer0}},
        {{launch_gemm_inst_ps0_out0_outer1, launch_gemm_inst_ps0_out1_outer1, launch_gemm_inst_ps0_out2_outer1},
         {launch_gemm_inst_ps1_out0_outer1, launch_gemm_inst_ps1_out1_outer1, launch_gemm_inst_ps1_out2_outer1}}};
    static const InstFn kws[2][3] = {{launch_gemm_kw_out0_outer0, launch_gemm_kw_out1_outer0, launch_gemm_kw_out2_outer0},
                                     {launch_gemm_kw_out0_outer1, launch_gemm_kw_out1_outer1, launch_gemm_kw_out2_outer1}};
    return (kw ? kws[outer ? 1 : 0][kind] : inst[outer ? 1 : 0][ps ? 1 : 0][kind])(tile, g, grid, st);
}

hipError_t launch_tiles(int tile, int outer, bool ps, bool out_f32, bool kw, const GemmGroup &g, dim3 grid, hipStream_t st)
{
    typedef hipError_t (*InstFn)(int, const GemmGroup &, dim3, hipStream_t);
    static const InstFn inst[2][2][2] = {{{launch_gemm_inst_ps0_out0_outer0, launch_gemm_inst_ps0_out1_outer0},
                                          {launch_gemm_inst_ps1_out0_outer0, launch_gemm_inst_ps1_out1_outer0}},
                                         {{launch_gemm_inst_ps0_out0_outer1, launch_gemm_inst_ps0_out1_outer1},
                                          {launch_gemm_inst_ps1_out0_outer1, launch_gemm_inst_ps1_out1_outer1}}};
    static const InstFn kws[2][2] = {{launch_gemm_kw_out0_outer0, launch_gemm_kw_out1_outer0}, {launch_gemm_kw_out0_outer1, launch_gemm_kw_out1_outer1}};
    return (kw ? kws[outer ? 1 : 0][out_f32] : inst[outer ? 1 : 0][ps][out_f32])(tile, g, grid, st);
}

// The tile of a product launched alone whose operands are blocked along K and carry 1 x 128 outer blocks.  The planned costs are those of row-major
// operands; with blocked ones two 128 x 128 workgroups on a CU are faster than every 256 x 128 and 128 x 256 tile that those costs choose for a product in one piece (they are
// chosen only where there are more 128 x 128 tiles than CUs).  Partial sums of a split keep the planned tile.  All these tiles add in the same order.
// us of the product, M x N x K, row-major on the planned 256 x 128 tile -> blocked on 128 x 128: 8192 x 3072 x 768 56.3 -> 53.1, 16384 x 8192 x 1024 354.6 -> 332.6,
// 6144 x 6144 x 1024 110.6 -> 93.3, 4096 x 2048 x 2048 44.6 -> 42.7, 9984 x 7936 x 256 82.5 -> 70.7, 9088 x 2944 x 768 72.2 -> 55.9, 5504 x 1024 x 256 11.6 -> 10.6; on a planned
// 128 x 256 one: 3456 x 12032 x 1024 115.4 -> 103.0, 640 x 11264 x 768 20.8 -> 20.0.  Where the tile stays 128 x 128, the layout alone gives 1.07 (8192 x 4096 x 4096 337 -> 315).
int tile_of_blocked(const Plan &p) { return p.split == 1 && !p.kw && (p.tile == 1 || p.tile == 2) ? 3 : p.tile; }

// Whether the plan's launch can read operands that are blocked along K (the reasons are at GroupPlan).
bool takes_blocked(const Plan &p, int64_t M, int64_t N, int64_t K, int outer)
{
    return M <= kMaxBlockedRows && N <= kMaxBlockedRows && !p.kw && (outer ? K % 256 == 0 : p.split == 1 || p.chunks_per_split % 2 == 0);
}

// Whether blocked operands pay for a product launched alone.  us of calls (quantizers and product), row-major -> blocked; runs of one side differ by up to 2 %:
// - Outer blocks, dX (rowwise: A comes from the row-wise quantizer, which takes 0.5 us more until it fills the chip): not for short reductions
//   (1792 x 256 x 256 13.4 -> 14.2, 512 x 6656 x 1280 33.2 -> 34.0, 7680 x 2304 x 256 37.0 -> 37.8), but from 2^21 elements of dY on (15616 x 128 -> 512 fused 59.7 -> 57.1), from
//   2^33 multiplications on (2048 x 5632 x 1536 68.7 -> 67.3; 512 x 7040 x 1792 with 2^32.6 43.2 -> 44.5), for long reductions (256 x 128 x 2816 26.5 -> 25.7; x 1536 22.2 -> 22.4),
//   and where the tile changes to 128 x 128.  dW: 0.2 us lost where the tile has 64 rows (256 x 2048 x 256 14.2 -> 14.5), else level or better (2048 x 1152 x 1024 30.0 -> 29.8).
// - Per-tensor scales: a row of up to 128 k is one stage's copy in either layout (65536 x 256 x 64 fused 86.3 -> 87.9, x 128 dX alone 33.3 -> 36.5), and 192 gains nothing
//   (4672 x 4736 x 192 38.6 -> 39.4).  Where the row-wise quantizer runs by itself (rowwise; the call for both gradients quantizes dY once for both), its tiles of 256 or 512
//   columns are part empty for short reductions (32768 x 256 x 320 35.1 -> 36.7; 16384 x 512 x 576 38.2 -> 37.3), and slivers of an output lose to its longer start (1024 x 64 x 768
//   23.5 -> 24.0).
bool blocked_pays(const Plan &p, int64_t M, int64_t N, int64_t K, int outer, bool rowwise)
{
    if (!outer) return rowwise ? K >= 512 && M >= 128 && N >= 128 : K >= 256;
    return K >= 2048 || (double)M * (double)N * (double)K >= 0x1p33 || tile_of_blocked(p) != p.tile || (rowwise ? M * K >= ((int64_t)1 << 21) : p.tile < 5);
}

// Operands in a layout that the launch would read as another one are refused: the product would be wrong without an error.
bool layout_fits(const Plan &p, const GemmOperand &A, const GemmOperand &B, int64_t K)
{
    return A.blocked == B.blocked && (!A.blocked || takes_blocked(p, A.rows, B.rows, K, A.outer));
}

hipError_t launch_planned(const Plan &plan, const GemmOperand &A, const GemmOperand &B, int64_t K, void *out, int out_f32, void *ws,
                          size_t ws_bytes, hipStream_t st)
{
    const int64_t M = A.rows, N = B.rows;
    if (!layout_fits(plan, A, B, K)) return hipErrorInvalidValue;
    Plan p = plan;
    if (A.blocked && A.outer) p.tile = tile_of_blocked(plan);
    if (M == 0 || N == 0) return hipSuccess;
    if (K == 0) {
        const int64_t n16 = M * N * (out_f32 ? 2 : 1);
        const int64_t want = (n16 + kThreads - 1) / kThreads;
        hipLaunchKernelGGL(zero_out_kernel, dim3((unsigned)(want > 4096 ? 4096 : want)), dim3(kThreads), 0, st,
                           static_cast<uint16_t *>(out), n16);
        return hipGetLastError();
    }
    const int outer = A.outer;
    if (p.split > 1 && (ws == nullptr || ws_bytes < (size_t)p.split * M * N * sizeof(float))) return hipErrorInvalidValue;
    const int64_t chunks = K / 64;
    const int split = p.split > 1 ? (int)((chunks + p.chunks_per_split - 1) / p.chunks_per_split) : 1;
    const GemmArgs g = args_of(A, B, K, split > 1 ? ws : out, out_f32, p.tile, p.chunks_per_split);
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n), 1, (unsigned)split);
    hipError_t e = launch_tiles(p.tile, outer, K % 256 == 0 && p.chunks_per_split % 4 == 0, split > 1 ? 2 : (out_f32 ? 1 : 0),
                                p.kw, g, grid, st);
    if (e != hipSuccess) return e;
    if (split > 1) {
        const int64_t mn = M * N;
        const unsigned rgrid = (unsigned)((mn + (int64_t)kThreads * 4 - 1) / ((int64_t)kThreads * 4));
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(rgrid), dim3(kThreads), 0, st,
                           reinterpret_cast<const float *>(ws), split, mn, A.gscale, B.gscale, outer, out, out_f32);
        e = hipGetLastError();
    }
    return e;
}

// Products in one launch.  Alone, each of them ends with a round of workgroups that leaves CUs idle (928 tiles on 512 places: the
// second round fills four fifths of them), and the next waits for its last one; together they share the last round.  They keep
// their own plans' order of summation - the reduction in one piece, by the same kernel, whose tiles all add in the same order -
// so that their bits do not depend on what is launched with them.  (The third, the outlier channels' part of dX, exists in no
// other call: it takes the kernel of the other two.)
//
// A launch together is taken where its estimate is below a share of the sum of the separate ones (0.95, see the sizes below).  Measured on 1965
// random layers, device time of the whole backward call against the separate launches: the 1600 that are joined run 1.07 to 1.25 times as fast,
// by tile, 15 of them slower (0.92 to 0.995: long reductions on 256-row tiles).
// - Split waves with per-tensor scales, 64 x 64 up to the four rounds that a product alone may have, and 128 x 128: 1.12 to 1.22, while the
//   estimate is 8 % too high in the median.  1.03 of the separate time is enough there (81 layers between 0.95 and 1.03: 1.10, eight of them
//   slower, 0.94 at worst; with more rounds of 64 x 64, 11200 x 448 -> 7936 in 2093 workgroups, 0.95).
// - Outer blocks: 128 x 128 takes 6 % less than its estimate in the median (which slows the workgroups of the last round as if each still shared
//   its CU), and is preferred at 0.95 of it (3 % and 5 % more than their estimate with 128 x 256 and 256 x 128).
// - Outer blocks, 256 x 128 and 128 x 256, one workgroup per CU: down to 0.86 where the second round was nearly full.  Workgroups are dealt in
//   turn over the XCDs and, inside each, over its four shader engines, and one that is due on an engine full of long ones waits although another has
//   room.  896 x 4352 -> 1664 has 136 long ones (35 us) and 238 short (21), which one pool of 256 places would finish in 41 us: workgroups that only
//   wait for these times take 57, and 43 with 119 and 221.  Up to three rounds these tiles must not be 5 % slower than the separate launches in the
//   pool of one engine's 8 CUs.
constexpr int kDealGroups = 32;

// When the last of the workgroups ends: count[i] of time[i] each, taken in order by `places` places.
double time_of_pool(const int64_t *count, const double *time, int n, int64_t places_all)
{
    double at[64], end = 0.0;                              // places and when they fall free, the earliest first
    int64_t places[64];
    int classes = 1;
    at[0] = 0.0;
    places[0] = places_all;
    for (int i = 0; i < n; ++i) {
        for (int64_t left = count[i]; left > 0;) {
            if (classes >= 63) return 1e300;
            const int64_t take = left < places[0] ? left : places[0];
            const double until = at[0] + time[i];
            left -= take;
            places[0] -= take;
            if (places[0] == 0) {
                for (int c = 1; c < classes; ++c) { at[c - 1] = at[c]; places[c - 1] = places[c]; }
                --classes;
            }
            int c = classes++;
            for (; c > 0 && at[c - 1] > until; --c) { at[c] = at[c - 1]; places[c] = places[c - 1]; }
            at[c] = until;
            places[c] = take;
            end = end < until ? until : end;
        }
    }
    return end;
}

// product of K in the launch together, as a plan
Plan joint_part(const GroupPlan &g, int64_t K) { return Plan{g.tile, 1, (int)(K / 64), g.kw, 0.0}; }

// Fills in the launch together of g's products, if there is one.
void plan_joint(GroupPlan &g, const int64_t (*mnk)[3], int outer)
{
    const int n = g.n;
    bool ps = true, whole = true;
    double apart = 0.0;
    for (int i = 0; i < n; ++i) {
        const int64_t M = mnk[i][0], N = mnk[i][1], K = mnk[i][2];
        if (M < (i < 2 ? 128 : 1) || N < (i < 2 ? 128 : 1) || K < 256) return;
        ps = ps && K % 256 == 0;
        whole = whole && M % 64 == 0 && N % 64 == 0;
        const Plan &p = g.own[i];
        if (i < 2 && (p.split > 1 || p.kw != g.own[0].kw)) return;
        apart += p.time;
    }
    g.kw = g.own[0].kw;
    const bool kw = g.kw;
    for (int i = 1; i < n; ++i)                            // the longest reduction first
        for (int j = i; j > 0 && mnk[g.order[j]][2] > mnk[g.order[j - 1]][2]; --j) std::swap(g.order[j], g.order[j - 1]);
    const int64_t longest = mnk[g.order[0]][2];
    double best_t = 1e300;
    for (int t = 0; t < kNumTiles; ++t) {
        if ((t == 0 && outer) || (t == 7 && (outer || !whole)) || ((t == 4 || (t == 6 && !kw)) && !ps)) continue;
        if (t >= 5 && !kw && longest > 16 * 64 * kNC) continue;
        const TileCfg &cfg = (t == 5 || t == 6) && !(kw && whole) ? kSmallRagged[outer][t - 5] : kTilesFit[outer][t];
        const int64_t bm = 64 * kTiles[t].tm, bn = 64 * kTiles[t].tn;
        bool same = true;
        int64_t count[kMaxGroup], wgs = 0;
        for (int i = 0; i < n; ++i) {
            const int64_t *s = mnk[g.order[i]];
            same = same && waves_split_k(t, s[2] / 64, 0, outer) == kw;
            count[i] = ((s[0] + bm - 1) / bm) * ((s[1] + bn - 1) / bn);
            wgs += count[i];
        }
        if (!same) continue;
        const int64_t per_cu = (wgs + kNumCU - 1) / kNumCU, conc = per_cu < cfg.occupancy ? per_cu : cfg.occupancy;
        if (wgs > 16 * kNumCU * conc) continue;            // many rounds: the last one counts for little
        const double slow = conc == 1 ? 1.0 : conc > 2 ? 1.95 : t >= 5 && !kw ? 1.4 : outer ? 1.52 : 1.58;
        double time[kMaxGroup];
        for (int i = 0; i < n; ++i)
            time[i] = ((double)((mnk[g.order[i]][2] / 64 + kNC - 1) / kNC) * cfg.t_stage + cfg.t_fixed) * slow;
        const bool sure = kw && !outer && (t == 7 || (t == 5 && wgs <= 4 * 2 * kNumCU));
        const double end = time_of_pool(count, time, n, kNumCU * conc), rank = outer && t == 3 ? 0.95 * end : end;
        if (end >= apart * (sure ? 1.03 : 0.95) || rank >= best_t) continue;
        if (outer && (t == 1 || t == 2) && wgs <= 3 * kNumCU) {
            for (int i = 0; i < n; ++i) count[i] = (count[i] + kDealGroups - 1) / kDealGroups;
            if (time_of_pool(count, time, n, kNumCU / kDealGroups * conc) >= 1.05 * apart) continue;
        }
        best_t = rank;
        g.tile = t;
    }
}

}  // namespace

GroupPlan plan_group(const int64_t (*mnk)[3], int n, int outer, bool rowwise)
{
    GroupPlan g{};
    g.n = n;
    g.tile = -1;
    for (int i = 0; i < n; ++i) {
        const int64_t M = mnk[i][0], N = mnk[i][1], K = mnk[i][2];
        g.order[i] = i;
        g.own[i] = make_plan(M, N, K, outer);
        g.blocked[i] = takes_blocked(g.own[i], M, N, K, outer);
        g.pays[i] = blocked_pays(g.own[i], M, N, K, outer, rowwise && i == 0);
        const size_t ws = split_bytes(g.own[i], M, N);
        g.ws = g.ws > ws ? g.ws : ws;
    }
    if (n > 1) plan_joint(g, mnk, outer);
    if (g.tile >= 0) {
        // outer blocks: as for a product alone, but the gain begins earlier (together 256 x 2944 -> 512 26.0 -> 26.3 us, 256 x 7808 -> 512 32.9 -> 32.3, 1280 x 2688 -> 1280 49.0 -> 47.9)
        bool all = true;
        double work = 0.0;
        for (int i = 0; i < n; ++i) {
            all = all && takes_blocked(joint_part(g, mnk[i][2]), mnk[i][0], mnk[i][1], mnk[i][2], outer);
            work += (double)mnk[i][0] * (double)mnk[i][1] * (double)mnk[i][2];
        }
        for (int i = 0; i < n; ++i) {
            g.blocked[i] = all;
            g.pays[i] = !outer || work >= 1.5e9;
        }
    }
    return g;
}

void planned_launch(const GroupPlan &plan, int i, const int64_t *mnk, int blocked, int outer, int *bm, int *bn, int *split, int *split_waves)
{
    const bool joint = plan.tile >= 0;
    const int t = joint ? plan.tile : blocked && outer ? tile_of_blocked(plan.own[i]) : plan.own[i].tile;
    *bm = 64 * kTiles[t].tm;
    *bn = 64 * kTiles[t].tn;
    *split = joint ? 1 : plan.own[i].split;
    *split_waves = joint ? plan.kw : plan.own[i].kw;
}

hipError_t launch_gemm_group(const GroupPlan &plan, const GemmProduct *p, int out_f32, void *ws, size_t ws_bytes, hipStream_t st)
{
    const int n = plan.n, outer = p[0].A.outer;
    // all of them before the first launch; one kernel reads the operands of a launch together
    for (int i = 0; i < n; ++i) {
        const bool alike = plan.tile < 0 || p[i].A.blocked == p[0].A.blocked;
        if (!alike || !layout_fits(plan.tile < 0 ? plan.own[i] : joint_part(plan, p[i].K), p[i].A, p[i].B, p[i].K)) return hipErrorInvalidValue;
    }
    if (plan.tile < 0) {
        for (int i = 0; i < n; ++i) {
            const hipError_t e = launch_planned(plan.own[i], p[i].A, p[i].B, p[i].K, p[i].out, out_f32, ws, ws_bytes, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    GemmGroup g;
    int wgs = 0;
    bool ps = true;
    for (int i = 0; i < kMaxGroup; ++i) {
        const GemmProduct &q = p[plan.order[i < n ? i : 0]];
        g.g[i] = args_of(q.A, q.B, q.K, q.out, out_f32, plan.tile, (int)(q.K / 64));
        g.first[i] = i < n ? wgs : INT_MAX;
        if (i < n) wgs += g.g[i].tiles_m * g.g[i].tiles_n;
        ps = ps && q.K % 256 == 0;
    }
    return launch_tiles(plan.tile, outer, ps, out_f32 != 0, plan.kw, g, dim3((unsigned)wgs, 1, 1), st);
}

void gemm_plan(int64_t M, int64_t N, int64_t K, int outer, int *bm, int *bn, int *split, int *split_waves)
{
    const Plan p = make_plan(M, N, K, outer);
    *bm = 64 * kTiles[p.tile].tm;
    *bn = 64 * kTiles[p.tile].tn;
    *split = p.split;
    *split_waves = p.kw ? 1 : 0;
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K, int outer)
{
    return split_bytes(make_plan(M, N, K, outer), M, N);
}

hipError_t launch_gemm_nt(const GemmOperand &A, const GemmOperand &B, int64_t K, void *out, int out_f32,
                          void *ws, size_t ws_bytes, hipStream_t st)
{
    return launch_planned(make_plan(A.rows, B.rows, K, A.outer), A, B, K, out, out_f32, ws, ws_bytes, st);
}

}  // namespace tj
