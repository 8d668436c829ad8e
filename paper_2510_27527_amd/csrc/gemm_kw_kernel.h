// The NT product on two packed NVFP4 operands for outputs too small to fill the chip: a workgroup's four waves split the
// reduction instead of the output tile.
//
// In gemm_nt_kernel a 64 x 64 tile gives each wave one 32 x 32 accumulator tile, and every MFMA pays for the expansion of two
// fragments (24 vector instructions): with one workgroup per CU the time is that instruction stream, K / 128 stages in
// a row, with a barrier in each.  Here every wave computes the whole TM x TN tiles of 32 x 32 of the workgroup for every fourth
// 64-k chunk (or 128-k outer block), so that an MFMA pays for (TM + TN) / (TM TN) fragments, and the waves meet only once,
// to add their four partial sums through LDS in a fixed order.
// Before (gemm_nt_kernel's tile of that output) and after, in us: 1024 x 1024 x 1024 8.6 -> 6.5, x 2048 13.6 -> 8.9 (64 x 64);
// 704 x 832 x 1600 11.7 -> 8.9; 640 x 1536 x 2496 22.2 (split over workgroups) -> 12.1; 2752 x 1088 x 4416 41.5 -> 33.5 (128 x 128);
// 3072 x 768 x 8192 54.4 (split) -> 48.6; outer blocks 1024 x 384 x 1024 10.5 -> 8.7, 1024 x 1024 x 1152 8.5.
// Bound now by the vector ALU (64 x 64: 12 of 16 instructions per MFMA are the expansion).  With 128 x 128 tiles counters show 5.0 to 5.6 vector
// instructions per MFMA and the matrix pipes busy 60 % of the time on the CUs that have a workgroup (768 x 3072 x 8192, 144 of them; 50 % with 198,
// 2752 x 1088 x 4416): a stage takes longer the more CUs draw on the L2 caches (0.64 us with 144, 0.8 with 256), and the closing sums 1.7 us.
//
// A pipeline stage is 256 k (512 with 1 x 128 outer blocks, a block per wave): 128 or 256 bytes of a row's codes at a time, whole
// cache lines, copied global -> LDS directly, two stages ahead in a ring of three (64 x 128 with outer blocks: one ahead in a ring
// of two); one barrier per stage.  (With a ring per wave, and 32 bytes of codes and 4 scale bytes per row and copy, the same
// kernel needed no barrier and was bound by the cache lines that each such piece drags in: 2048 x 2048 x 4096 40.9 us against 32.3, 2752 x 1088 x 4416 41.4 against 33.5.)
//   codes : 16-byte slot of (row, piece p) = row * SLOTS + (p ^ swz(row)), so that 16 consecutive rows cover 16 different 16-byte
//           columns of the 256-byte bank row
//   scales: 4 bytes per chunk, [row][chunk of the stage].  A row's last stage that is not whole is fetched from the row's last
//           bytes and lands as many bytes earlier, over the unused end of the previous row's, so that nothing past a row is
//           read.  (A row has at least one whole stage's scales: the launcher takes this kernel from K = 256 / 768 on.)
//   OUTER : one float per row, [block of the stage][row], in a ring of four stages
// Rows past M / N read the operand's last row and are never stored; chunks past the end of K count with zero scales.
#pragma once
#include "gemm_kernel.h"

namespace tj {

namespace {

constexpr int vm_wait(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }   // s_waitcnt immediate: vmcnt(n) and nothing else

template <int TM, int TN, int OUTER>
struct KwShape {
    static constexpr int ROWS = 32 * (TM + TN);
    static constexpr int NCW = OUTER ? 2 : 1;                        // chunks of a stage per wave
    static constexpr int SLOTS = 8 * NCW;                            // 16-byte pieces per row and stage
    static constexpr int D = OUTER && ROWS > 128 ? 2 : 3;            // stages in the ring
    static constexpr int CODE = ROWS * SLOTS * 16, SC_ROW = 16 * NCW, SC = 32 + ROWS * SC_ROW, GS = OUTER ? 4 * ROWS * 4 : 0;
    static constexpr int RING = D * (CODE + SC) + 4 * GS;
    static constexpr int PHASES = TM * TN / 4;                       // of the closing reduction, 64 KB each
    static constexpr int RED = (PHASES > 1 ? 2 : 1) * 65536;
    static constexpr int LDS = RING > RED ? RING : RED;
};

template <int TM, int TN, int OUT, int OUTER, class Args>   // OUT: 0 bf16, 1 f32, 2 raw f32 split-K partial
__global__ __launch_bounds__(kThreads, (TM * TN == 4 ? 2 : 1)) void gemm_kw_kernel(Args args)
{
    typedef KwShape<TM, TN, OUTER> S;
    constexpr int BM = 32 * TM, BN = 32 * TN, ROWS = S::ROWS, D = S::D, NCW = S::NCW, SLOTS = S::SLOTS;
    constexpr int NC = 4 * NCW;                                      // chunks per stage
    constexpr int ROWS_I = 64 / SLOTS;                               // rows of one copy instruction
    constexpr int LC = ROWS * SLOTS / kThreads, LA = BM * SLOTS / kThreads;   // code copies per wave and stage (the first LA of A)
    constexpr int SROWS_I = 64 / NCW, LS = (ROWS / SROWS_I + 3) / 4; // scale copies: rows per instruction, copies per wave
    constexpr int LG = OUTER ? ROWS / 64 : 0;                        // outer scales of the wave's own block
    constexpr int NLOAD = LC + LS + LG;
    static_assert((D - 2) * NLOAD <= 63, "the waits count the newest D - 2 stages' copies");
    static_assert(BM * SLOTS % kThreads == 0 && BN * SLOTS % kThreads == 0 && BM % 64 == 0 && BN % 64 == 0, "whole copy instructions per operand");
    constexpr bool SWAP = OUT == 0;
    constexpr int RM = TM / 2, RN = TN / 2;                          // tiles per wave after the reduction

    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, kg = lane >> 5;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem_raw;
    constexpr int SC_BASE = D * S::CODE + 32, GS_BASE = D * (S::CODE + S::SC);

    int tile_m, tile_n, wg;
    const GemmArgs &g = product_of_workgroup(args, wg);
    tile_of_workgroup(g, wg, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int64_t cbeg = (int64_t)blockIdx.z * g.chunks_per_split;
    int64_t cend = cbeg + g.chunks_per_split;
    if (cend > g.K / 64) cend = g.K / 64;
    const int nchunks = (int)(cend - cbeg);
    const int nk = (nchunks + NC - 1) / NC;

    float16_t acc[TM][TN];
    float16_t zero16;
#pragma unroll
    for (int e = 0; e < 16; ++e) zero16[e] = 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = zero16;
    float16_t part[TM][TN];                                          // OUTER: the running sum of the current 128-k block

    if (nchunks > 0) {
        const int64_t cstride = g.K / 2, sstride = g.K / 16, nkb = g.K >> 7;
        const int last_a = (int)((g.M - m0 < BM ? g.M - m0 : BM) - 1), last_b = (int)((g.N - n0 < BN ? g.N - n0 : BN) - 1);
        // tile row (A's, then B's) -> existing row of its operand, relative to the tile's first
        auto clamp_row = [&](int r) { return (uint32_t)(r < BM ? (r < last_a ? r : last_a) : (r - BM < last_b ? r - BM : last_b)); };
        uint32_t coff[LC], soff[LS], goff[OUTER ? LG : 1];           // byte offsets from the tile's (uniform) base pointers
        auto swz = [](int row) { return NCW == 1 ? (row >> 1) & 7 : row & 15; };
        const int piece0 = lane & (SLOTS - 1);
#pragma unroll
        for (int u = 0; u < LC; ++u) {
            const int row = (u * 4 + wave) * ROWS_I + lane / SLOTS;
            coff[u] = clamp_row(row) * (uint32_t)cstride + 16u * (piece0 ^ swz(row));
        }
#pragma unroll
        for (int u = 0; u < LS; ++u) {
            const int row = ((u * 4 + wave) * SROWS_I) % ROWS + lane / NCW;
            soff[u] = clamp_row(row) * (uint32_t)sstride + 16u * (lane % NCW);
        }
        if (OUTER)
#pragma unroll
            for (int u = 0; u < LG; ++u) goff[u] = clamp_row(u * 64 + lane) * (uint32_t)nkb * 4u;
        const uint8_t *a_cbase = g.a_codes + m0 * cstride + cbeg * 32, *b_cbase = g.b_codes + n0 * cstride + cbeg * 32;
        const uint8_t *a_sbase = g.a_scales + m0 * sstride + cbeg * 4, *b_sbase = g.b_scales + n0 * sstride + cbeg * 4;
        const float *a_gbase = OUTER ? g.a_gscale + m0 * nkb + (cbeg >> 1) : nullptr;
        const float *b_gbase = OUTER ? g.b_gscale + n0 * nkb + (cbeg >> 1) : nullptr;
        const int last_start = (int)(sstride - S::SC_ROW - cbeg * 4);   // of a row's last stage of scales

        // All copies of stage kt into ring slot `slot`.  The waits count them, so a stage past the end and pieces past the last chunk are
        // copied too (never used), from the first bytes of the tile: one cache line for a whole instruction.
        auto issue = [&](int kt, int slot) {
            const bool stage_ok = kt < nk;
            const int c0 = stage_ok ? kt * NC : 0, have = stage_ok ? nchunks - c0 : 0;
            const uint8_t *ac = a_cbase + (int64_t)c0 * 32, *bc = b_cbase + (int64_t)c0 * 32;
            const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + slot * S::CODE + wave * 1024);
            if (have >= NC) {
#pragma unroll
                for (int u = 0; u < LC; ++u) lds_dma16(u < LA ? ac : bc, coff[u], dst + u * 4096);
            } else {
#pragma unroll
                for (int u = 0; u < LC; ++u) {
                    const int p = piece0 ^ swz((u * 4 + wave) * ROWS_I + lane / SLOTS);
                    lds_dma16(u < LA ? ac : bc, p < 2 * have ? coff[u] : 0u, dst + u * 4096);
                }
            }
            const uint32_t used = stage_ok ? 0xFFFFFFFFu : 0u;
            const int start = kt * S::SC_ROW < last_start ? kt * S::SC_ROW : last_start;
            const int back = -start & (S::SC_ROW - 1);
#pragma unroll
            for (int u = 0; u < LS; ++u) {
                const int row0 = ((u * 4 + wave) * SROWS_I) % ROWS;
                lds_dma16((row0 < BM ? a_sbase : b_sbase) + start, soff[u] & used, lds_base + SC_BASE + slot * S::SC + row0 * S::SC_ROW - back);
            }
            if (OUTER) {
                int kb = (c0 >> 1) + wave;
                if (kb * 2 >= nchunks) kb = 0;
#pragma unroll
                for (int u = 0; u < LG; ++u)
                    lds_dma4((u < BM / 64 ? a_gbase : b_gbase) + kb, goff[u] & used, lds_base + GS_BASE + (kt & 3) * S::GS + (wave * ROWS + u * 64) * 4);
            }
        };
        struct Raw { uint4 qa[TM], qb[TN]; };                        // 32 codes per fragment
        uint32_t scA[NCW][TM], scB[NCW][TN];                         // four scale bytes per chunk and fragment row
        auto read_raw = [&](Raw &r, int slot, int c) {
            const uint4 *codes = reinterpret_cast<const uint4 *>(smem_raw + slot * S::CODE);
            const int p = 2 * (wave * NCW + c) + kg;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = i * 32 + lr;
                r.qa[i] = codes[row * SLOTS + (p ^ swz(row))];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = BM + j * 32 + lr;
                r.qb[j] = codes[row * SLOTS + (p ^ swz(row))];
            }
        };
        auto read_scales = [&](int slot) {
            const uint8_t *sp = smem_raw + SC_BASE + slot * S::SC + wave * NCW * 4;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int c = 0; c < NCW; ++c) scA[c][i] = reinterpret_cast<const uint32_t *>(sp + (i * 32 + lr) * S::SC_ROW)[c];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int c = 0; c < NCW; ++c) scB[c][j] = reinterpret_cast<const uint32_t *>(sp + (BM + j * 32 + lr) * S::SC_ROW)[c];
        };
        // scale factors of a chunk's two groups per lane, as in gemm_nt_kernel; a stage past the wave's last chunk gets zeros, by a
        // selector of zero bytes or a field width of 0
        constexpr bool PAIR = TM * TN <= 6;
        uint32_t sc_sel = kg ? 0x0C030C02u : 0x0C010C00u, width = 8;
        half2_t fA[TM], fB[TN];
        auto factor = [&](uint32_t sc, int ks) {
            if (PAIR) return __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(0u, sc, sc_sel) << 7);
            return scale_pair(__builtin_amdgcn_ubfe(sc, 16 * kg + 4 * ks, width));
        };
        auto half_of = [&](half2_t f, int ks) { return !PAIR ? f : ks < 2 ? (half2_t){f.x, f.x} : (half2_t){f.y, f.y}; };
        struct Ops { half8_t a[TM], b[TN]; };
        auto expand = [&](Ops &o, const Raw &r, int c, int ks) {
            if (ks == 0 || (!PAIR && ks == 2)) {
#pragma unroll
                for (int i = 0; i < TM; ++i) fA[i] = factor(scA[c][i], ks);
#pragma unroll
                for (int j = 0; j < TN; ++j) fB[j] = factor(scB[c][j], ks);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) o.a[i] = expand8(pick(r.qa[i], ks), half_of(fA[i], ks));
#pragma unroll
            for (int j = 0; j < TN; ++j) o.b[j] = expand8(pick(r.qb[j], ks), half_of(fB[j], ks));
        };
        auto zero_if_past = [&](int kt) {
            if (kt * NC + wave * NCW >= nchunks) { sc_sel = 0x0C0C0C0Cu; width = 0; }
        };

        // (the 4 x 4 tiles have no registers for two sets of raw codes: theirs are fetched in the stage's last step)
        constexpr bool ONE = TM * TN == 16;
        constexpr int FETCH = ONE ? 4 * NCW - 1 : 4 * NCW - 2;      // the step in which the next stage's first fragments are fetched
        Raw raw[ONE ? 1 : 2];
        Ops op[2];
        issue(0, 0);
        if (D > 2) issue(1, 1);
        __builtin_amdgcn_s_waitcnt(vm_wait((D - 2) * NLOAD));        // stage 0 has landed
        __syncthreads();
        zero_if_past(0);
        read_scales(0);
        read_raw(raw[0], 0, 0);
        expand(op[0], raw[0], 0, 0);

        int slot = 0;
        constexpr int STEPS = 4 * NCW;
        auto stage = [&](int kt, auto par) {
            constexpr int P = decltype(par)::value;                  // raw[P] holds the stage's first chunk
            const int next = slot == D - 1 ? 0 : slot + 1;
            if (D > 2) issue(kt + 2, slot == 0 ? D - 1 : slot - 1);
            else issue(kt + 1, next);
#pragma unroll
            for (int gs = 0; gs < STEPS; ++gs) {
                const int c = gs / 4, ks = gs % 4;
                if (ks == 1 && c + 1 < NCW) read_raw(raw[P ^ 1], slot, c + 1);
                if (gs == FETCH) {
                    __builtin_amdgcn_s_waitcnt(vm_wait((D - 2) * NLOAD));   // all but the newest D - 2 stages' copies: stage kt + 1 has landed
                    __syncthreads();
                    zero_if_past(kt + 1);
                    read_scales(next);
                    read_raw(raw[NCW == 2 || ONE ? P : P ^ 1], next, 0);
                }
                if (gs + 1 < STEPS) expand(op[(gs + 1) & 1], raw[P ^ ((gs + 1) / 4)], (gs + 1) / 4, (gs + 1) % 4);
                else expand(op[0], raw[NCW == 2 || ONE ? P : P ^ 1], 0, 0);
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        float16_t &dst = OUTER ? part[a][b] : acc[a][b];
                        const float16_t addend = (OUTER && gs == 0) ? zero16 : dst;
                        dst = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_f16(op[gs & 1].b[b], op[gs & 1].a[a], addend, 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_32x32x16_f16(op[gs & 1].a[a], op[gs & 1].b[b], addend, 0, 0, 0);
                    }
                // issue order: one MFMA, then (in the steps that fetch raw fragments) two LDS reads, then its share of the expansion
#pragma unroll
                for (int q = 0; q < TM * TN; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (((ks == 1 && c + 1 < NCW) || gs == FETCH) && q < TM + TN) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, (8 * (TM + TN) + TM * TN - 1) / (TM * TN) + 1, 0);
                }
            }
            if (OUTER && kt * NC + wave * NCW < nchunks) {
                // end of the wave's outer block: total += block sum * S_A[m] * S_B[n], as in gemm_nt_kernel.  A wave without a block in the
                // last stage adds nothing: the scales in its place are another block's, and an infinite one would make its zero sum a NaN.
                const float *gsr = reinterpret_cast<const float *>(smem_raw + GS_BASE + (kt & 3) * S::GS) + wave * ROWS;
                rescale_add<TM, TN, SWAP>(acc, part, gsr, gsr + BM, lr, kg);
            }
            slot = next;
        };
        if constexpr (NCW == 2 || ONE) {
            for (int kt = 0; kt < nk; ++kt) stage(kt, std::integral_constant<int, 0>{});
        } else {
            for (int kt = 0; kt < nk; kt += 2) {
                stage(kt, std::integral_constant<int, 0>{});
                if (kt + 1 >= nk) break;
                stage(kt + 1, std::integral_constant<int, 1>{});
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);                          // drain the look-ahead copies before the LDS is reused
    }
    __syncthreads();

    // The four partial sums, tile by tile: in a phase every wave writes one tile of each quadrant and adds up its own quadrant's
    // from the four, in wave order.  Two buffers alternate, so one barrier per phase.
    const int wm = wave >> 1, wn = wave & 1;
    float16_t sum[RM][RN];
#pragma unroll
    for (int ri = 0; ri < RM; ++ri)
#pragma unroll
        for (int rj = 0; rj < RN; ++rj) {
            uint8_t *buf = smem_raw + ((ri * RN + rj) & 1) * (S::PHASES > 1 ? 65536 : 0);
#pragma unroll
            for (int qm = 0; qm < 2; ++qm)
#pragma unroll
                for (int qn = 0; qn < 2; ++qn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float16_t &t = acc[qm * RM + ri][qn * RN + rj];
                        *reinterpret_cast<float4 *>(buf + ((qm * 2 + qn) * 4 + wave) * 4096 + q * 1024 + lane * 16) =
                            make_float4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
                    }
            __syncthreads();
            const uint8_t *own = buf + wave * 4 * 4096 + lane * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4 s = *reinterpret_cast<const float4 *>(own + q * 1024);
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float4 t = *reinterpret_cast<const float4 *>(own + w * 4096 + q * 1024);
                    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
                }
                sum[ri][rj][4 * q] = s.x; sum[ri][rj][4 * q + 1] = s.y; sum[ri][rj][4 * q + 2] = s.z; sum[ri][rj][4 * q + 3] = s.w;
            }
        }
    if (SWAP) __syncthreads();                                       // the epilogue stages its rows in the same LDS
    store_tile<RM, RN, OUT, SWAP, OUTER>(sum, g, m0, n0, wm, wn, lr, kg, smem_raw);
}

template <int TM, int TN, int OUT, int OUTER, class Args>
hipError_t launch_kw_cfg(const Args &g, dim3 grid, hipStream_t st)
{
    constexpr int lds = KwShape<TM, TN, OUTER>::LDS;
    static_assert(lds <= 160 * 1024, "LDS of one CU");
    auto kern = gemm_kw_kernel<TM, TN, OUT, OUTER, Args>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, st, g);
    return hipGetLastError();
}

// tile: 5 64x64, 6 64x128, 7 128x128 (tensor mode only, never split over workgroups)
template <int OUT, int OUTER, class Args>
hipError_t launch_kw_tile(int tile, const Args &g, dim3 grid, hipStream_t st)
{
    switch (tile) {
        case 5: return launch_kw_cfg<2, 2, OUT, OUTER>(g, grid, st);
        case 6: return launch_kw_cfg<2, 4, OUT, OUTER>(g, grid, st);
        default:
            if constexpr (OUTER == 0 && OUT != 2) return launch_kw_cfg<4, 4, OUT, 0>(g, grid, st);
            else return hipErrorInvalidValue;
    }
}

}  // namespace

}  // namespace tj
