// OsciReset kernels (TetraJet-v2 Sec. 3.2-3.3: Alg. 1 OscillationSuppress; Appendix Alg. 2 UpdateOscillationStats and
// Alg. 3, its memory-efficient form that tracks only the k weights closest to a rounding threshold)
// for one weight matrix of binary32 master weights [C x D].  Q(W) is the forward weight quantizer - groups of 16 along
// D, round-to-nearest, nearest-even E4M3 scales, 1 x 128 FP32 outer blocks - followed by the binary32 dequantization
// (P * S_block) * S_global.  Both kernels are elementwise streams: a lane owns 8 consecutive weights (two 128-bit
// loads per array), two lanes a group of 16, sixteen lanes an outer block; maxima travel by DPP.
#include <type_traits>

#include "device_fmt.h"
#include "internal.h"
#include "osci_search.h"

namespace tj {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxCountingWgs = 256;      // workgroups of a reset that counts: each ends with an addition to one counter

struct F8 { float v[8]; };

__device__ __forceinline__ F8 load8(const float *p)
{
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    return F8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ __forceinline__ void store8(float *p, const F8 &x)
{
    *reinterpret_cast<float4 *>(p) = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
    *reinterpret_cast<float4 *>(p + 4) = make_float4(x.v[4], x.v[5], x.v[6], x.v[7]);
}

// The lane's 8 weights quantized; all 16 lanes of the outer block must be active.
struct Quant8 {
    uint32_t codes;      // eight E2M1 codes
    uint32_t top;        // pattern of the largest magnitude of the lane's weights
    float sb, S_g;       // block and outer scale
};
__device__ __forceinline__ Quant8 quantize8(const F8 &x, const float *inv_tab)
{
    uint32_t hm = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t ab = f2u(x.v[i]) & 0x7FFFFFFFu;
        hm = hm > ab ? hm : ab;
    }
    const uint32_t o1 = dpp<DPP_QUAD_XOR1>(hm);
    const uint32_t bm = hm > o1 ? hm : o1;                  // group of 16
    uint32_t gm = bm, t;
    t = dpp<DPP_QUAD_XOR2>(gm);       gm = gm > t ? gm : t;
    t = dpp<DPP_ROW_HALF_MIRROR>(gm); gm = gm > t ? gm : t;
    t = dpp<DPP_ROW_MIRROR>(gm);      gm = gm > t ? gm : t;  // outer block of 128
    const OuterScale os = outer_scale(u2f(gm));
    const uint32_t sc = e4m3_round<false>(u2f(bm) * os.inv_cg);
    const float r = os.inv_sg * inv_tab[sc];
    uint32_t codes = 0;
    codes = e2m1_rtn_pair<0>(codes, x.v[0] * r, x.v[1] * r);
    codes = e2m1_rtn_pair<1>(codes, x.v[2] * r, x.v[3] * r);
    codes = e2m1_rtn_pair<2>(codes, x.v[4] * r, x.v[5] * r);
    codes = e2m1_rtn_pair<3>(codes, x.v[6] * r, x.v[7] * r);
    return Quant8{codes, hm, e4m3_value(sc), os.S_g};
}
__device__ __forceinline__ F8 dequantize8(const Quant8 &k)
{
    const float2_t p0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(k.codes, 1.0f, 0) * k.sb;   // exact: 6 significant bits
    const float2_t p1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(k.codes, 1.0f, 1) * k.sb;
    const float2_t p2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(k.codes, 1.0f, 2) * k.sb;
    const float2_t p3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(k.codes, 1.0f, 3) * k.sb;
    return F8{{p0.x * k.S_g, p0.y * k.S_g, p1.x * k.S_g, p1.y * k.S_g, p2.x * k.S_g, p2.y * k.S_g, p3.x * k.S_g, p3.y * k.S_g}};
}
__device__ __forceinline__ F8 quant_dequant8(const F8 &x, const float *inv_tab) { return dequantize8(quantize8(x, inv_tab)); }

// nchunks = C * D / 8 is a multiple of 16 (D % 128 == 0), so a 16-lane row is either whole or absent
__global__ __launch_bounds__(kThreads) void osci_update_kernel(const float *W, float *W_prev, float *dist_m, float *dist_q,
                                                               int64_t nchunks, int first)
{
    __shared__ float inv_tab[128];
    fill_inv_table(inv_tab);
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c >= nchunks) return;
    const int64_t e = c * 8;
    const F8 w = load8(W + e);
    if (first) {
        const F8 z{{0, 0, 0, 0, 0, 0, 0, 0}};
        store8(W_prev + e, w);
        store8(dist_m + e, z);
        store8(dist_q + e, z);
        return;
    }
    const F8 wp = load8(W_prev + e);
    F8 dm = load8(dist_m + e), dq = load8(dist_q + e);
    const F8 q = quant_dequant8(w, inv_tab), qp = quant_dequant8(wp, inv_tab);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        dm.v[i] = dm.v[i] + fabsf(w.v[i] - wp.v[i]);
        dq.v[i] = dq.v[i] + fabsf(q.v[i] - qp.v[i]);
    }
    store8(W_prev + e, w);
    store8(dist_m + e, dm);
    store8(dist_q + e, dq);
}

__global__ __launch_bounds__(kThreads) void osci_suppress_kernel(float *W, const float *dist_m, const float *dist_q, float tau,
                                                                 int64_t nchunks, unsigned long long *n_reset)
{
    __shared__ float inv_tab[128];
    __shared__ unsigned int wg_count;
    fill_inv_table(inv_tab);
    if (threadIdx.x == 0) wg_count = 0;
    __syncthreads();
    unsigned int mine = 0;
    // Two chunks per thread and iteration, all their loads in flight together.  The counter is one address for the whole
    // chip, and additions to it are executed one after the other at about 10 ns each: with a workgroup per 256 chunks they
    // outlast the reading.  One workgroup per CU, one addition each, reads as fast as the other sizes of launch or faster.
    // Sources rotating through more than the last-level cache, at most 256 / 512 / 1024 / 4096 / any number of workgroups (us):
    // 3072 x 768 12.4 / 14.8 / 19.7 / 21.0 / 21.1, 8192 x 1024 30.9 / 31.8 / 33.6 / 58.0 / 58.0, 8192 x 4096 108 / 110 / 113 / 110 / 214,
    // 8192 x 8192 213 / 225 / 231 / 224 / 422, 16384 x 8192 421 / 459 / 481 / 462 / 835.  Without a counter a workgroup per 256
    // chunks is fastest: 8192 x 1024 27.4 us (256 workgroups 30.2), 8192 x 8192 207 (213).
    const int64_t stride = (int64_t)gridDim.x * kThreads;      // a multiple of 16: rows of 16 lanes stay whole
    for (int64_t c0 = (int64_t)blockIdx.x * kThreads + threadIdx.x; c0 < nchunks; c0 += 2 * stride) {
        F8 w[2], dm[2], dq[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t e = (u == 0 || c0 + stride < nchunks ? c0 + u * stride : c0) * 8;    // past the end: chunk c0 again, not used
            w[u] = load8(W + e);
            dm[u] = load8(dist_m + e);
            dq[u] = load8(dist_q + e);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t c = c0 + u * stride;
            if (c >= nchunks) break;
            const F8 q = quant_dequant8(w[u], inv_tab);
            unsigned int here = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float risk = dq[u].v[i] / dm[u].v[i];    // IEEE quotient; 0 / 0 is NaN and compares false
                if (risk >= tau) {
                    w[u].v[i] = q.v[i];
                    ++here;
                }
            }
            if (here) store8(W + c * 8, w[u]);
            mine += here;
        }
    }
    if (n_reset) {
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
        if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&wg_count, mine);
        __syncthreads();
        if (threadIdx.x == 0 && wg_count) atomicAdd(n_reset, (unsigned long long)wg_count);
    }
}

// ---- Appendix Alg. 3: selection of the k largest sensitivity scores (equal scores in ascending index order) ----------
//
// Scores are non-negative binary32 values, so they order like their bit patterns (a NaN counts as one value above
// infinity).  The k-th largest pattern is found by
// narrowing an interval [lo, lo + span) that holds it: a histogram pass over the tensor counts the patterns of the
// interval in bins (2048, then 32768), and the workgroup that finishes last picks the bin.  The first pass splits the patterns where
// scores live (|x - Q(x)| / binwidth is at most 1, and all but a few lie above 2^-8) into 256 bins per octave, with one
// open bin below and one above: 15 bits are left after it, none after the second pass.  (An equal
// split of all patterns put the scores of normal weights into a dozen bins, and their LDS counters became the bound: 76
// us for the first pass on 8192 x 1024, 19 us now.)  Only a threshold in an open bin needs the third pass; otherwise it
// ends at once.  The tensor is then compacted in index order: a count of (greater, equal) per 2048-element tile, whose
// last workgroup turns the counts into exclusive sums, and a pass that ranks every selected element and writes its index
// and the states of the tracked subset.  Every pass recomputes Q(W) (the scores are never stored: the point of the
// algorithm is to keep no per-element state).
//
// What workgroups leave for the last one travels by device-scope atomics (additions, stores, loads): they meet in
// memory, not in one of the eight L2 caches.
//
// Additions to one address are executed one after the other (about 8 ns each), so the passes that end with additions to
// shared counters run as at most kPassWgs workgroups of 1024 threads: 256 of them cost 2 us, 1024 of 256 threads 8 us.
//
// The sensitivity score of Appendix Alg. 3 is |x - Q(x)| / binwidth(Q(x)), binwidth = (length of the interval of scaled values
// that round to the code's magnitude) * RN(S_block * S_global); 0 in a block whose scale is 0.  Its correctly rounded quotient was
// a third of the passes' instructions, and the choice of the bin's length a fifth.  The passes therefore look at an estimate, num *
// rcp(unit) * (1 / bin), and take the quotient only where the estimate is within kNear patterns of a value at which their
// answer changes: a boundary between bins in the first pass (one chunk of 64 lanes in four), the interval that holds the
// threshold in a later one (these elements are put aside and divided at the end, all lanes busy), the threshold itself after
// that.  Error of the estimate, in units of 2^-24 relative: reciprocal 2, the two products 2, 4/3 and 2/3 rounded 1, the
// rounding of 0.75 * unit or 1.5 * unit 1, of the quotient 1; 7 in all, at most 7 patterns, 14 across a power of two.
// 8192 x 1024, 5 % selected: passes of 18.8, 15.8, 15.5, 4.6 (ends at once), 21.3 (count) and 17.4 us (emit) before; 14.3, 19.5, 4.5
// (ends at once), 17.3 and 14.2 with the estimate, the choice of the first bin in the second pass, and the rest of the interval
// resolved by that pass in 32768 bins.  Two chunks in flight per thread instead of one changed nothing: the passes wait for the
// vector ALU, not for memory.
constexpr int kTile = kThreads * 8;
constexpr int kPassThreads = 1024, kPassWgs = 256, kPassWaves = kPassThreads / 64;

struct SelState {
    SelInterval iv;       // the keys that hold the threshold
    uint32_t kneed;       // how many elements are still to be taken among those of the interval
    uint32_t thr;         // width 0: the key of the k-th largest score
    uint32_t ties;        // elements equal to thr that belong to the selection (the first ones in index order)
    uint32_t done[5];     // workgroups that have finished, per pass
};

__device__ __forceinline__ uint32_t load_dev(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_dev(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// true in every thread of the workgroup that arrives last; what the others sent by device-scope atomics before has landed
__device__ __forceinline__ bool last_to_arrive(uint32_t *counter, uint32_t *flag)
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");   // this wave's atomics have been executed
    __syncthreads();
    if (threadIdx.x == 0) *flag = atomicAdd(counter, 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    return *flag != 0;
}

__global__ __launch_bounds__(kThreads) void osci_zero_kernel(SelState *st, uint32_t *first, uint32_t *later)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < kFirstBins) first[i] = 0;
    else if (i < kFirstBins + kBins) later[i - kFirstBins] = 0;
    if (i < 5) st->done[i] = 0;
}

// 1 / bin, by the code's magnitude
__device__ __forceinline__ void fill_inv_bins(float *tab)
{
    if (threadIdx.x < 8) tab[threadIdx.x] = threadIdx.x < 4 ? 2.0f : threadIdx.x == 4 ? 4.0f / 3.0f : threadIdx.x == 6 ? 2.0f / 3.0f : 1.0f;
}
__device__ __forceinline__ float bin_width(uint32_t codes, int i, float unit)
{
    const uint32_t m = (codes >> (4 * i)) & 7u;
    return (m < 4 ? 0.5f : m == 4 ? 0.75f : m == 6 ? 1.5f : 1.0f) * unit;
}
__device__ __forceinline__ uint32_t score_bits(float num, float width) { return f2u(width == 0.0f ? 0.0f : num / width); }

// Patterns of the estimated scores of the lane's 8 weights, and the factors of the exact ones.  ok: the estimate holds - the unit is
// a normal number whose reciprocal is one too, and every weight of the lane is finite and at most 8 units (so is its
// distance from Q(x), and nothing overflows).
struct Scores8 {
    uint32_t p[8];
    F8 q, num;
    float unit;
    uint32_t codes;
    bool ok;
};
__device__ __forceinline__ Scores8 scores8(const F8 &x, const float *inv_tab, const float *inv_bins)
{
    Scores8 s;
    const Quant8 k = quantize8(x, inv_tab);
    s.q = dequantize8(k);
    s.codes = k.codes;
    s.unit = k.sb * k.S_g;
    const float y = __builtin_amdgcn_rcpf(s.unit);
    s.ok = s.unit > 0x1p-100f && s.unit < 0x1p100f && u2f(k.top) * y <= 8.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        s.num.v[i] = fabsf(x.v[i] - s.q.v[i]);
        s.p[i] = f2u(s.num.v[i] * y * inv_bins[(k.codes >> (4 * i)) & 7u]);
    }
    return s;
}
__device__ __forceinline__ uint32_t exact_score(const Scores8 &s, int i) { return score_bits(s.num.v[i], bin_width(s.codes, i, s.unit)); }

// exclusive prefix sum of v over the workgroup's threads (thread order) and their total; red: one word of LDS per wave
template <int WAVES>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *red, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    __syncthreads();                                       // the previous use of red is over
    if (lane == 63) red[wave] = incl;
    __syncthreads();
    uint32_t base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t r = red[w];
        base += w < wave ? r : 0u;
        total += r;
    }
    return base + incl - v;
}

// The bin, counted from the top, that holds the kneed-th key of the BINS counted in LDS, and the kneed that is left inside
// it; in every thread.  A thread's BINS / kPassThreads consecutive bins are read in rotated order, so that the lanes of a wave meet
// different banks.
template <int BINS>
__device__ __forceinline__ uint2 pick_bin(const uint32_t *bins, uint32_t *red, uint2 *picked, uint32_t kneed)
{
    constexpr int PER = BINS / kPassThreads;
    const uint32_t *own = bins + (kPassThreads - 1 - threadIdx.x) * PER;   // thread 0 holds the top ones
    uint32_t n = 0, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) n += own[(i + threadIdx.x) & (PER - 1)];
    uint32_t above = block_exclusive_scan<kPassWaves>(n, red, total);
    if (above < kneed && kneed <= above + n) {             // exactly one thread
        int i = PER - 1;
        while (kneed > above + own[i]) above += own[i--];  // ends at own[0] at the latest
        *picked = make_uint2((uint32_t)(own - bins + i), kneed - above);
    }
    __syncthreads();
    return *picked;
}

// The last workgroup's choice from the counts of all: read (all loads in flight together) and cleared for the next pass.
template <int BINS>
__device__ __forceinline__ uint2 pick_from_memory(uint32_t *hist, uint32_t *bins, uint32_t *red, uint2 *picked, uint32_t kneed)
{
    uint32_t n[BINS / kPassThreads];
#pragma unroll
    for (int u = 0; u < BINS / kPassThreads; ++u) n[u] = load_dev(&hist[u * kPassThreads + threadIdx.x]);
#pragma unroll
    for (int u = 0; u < BINS / kPassThreads; ++u) {
        bins[u * kPassThreads + threadIdx.x] = n[u];
        store_dev(&hist[u * kPassThreads + threadIdx.x], 0u);
    }
    __syncthreads();
    return pick_bin<BINS>(bins, red, picked, kneed);
}
__device__ __forceinline__ void store_interval(SelState *st, const SelInterval &iv, uint32_t kneed)
{
    if (threadIdx.x == 0) {
        st->iv = iv;
        st->thr = iv.lo;
        st->kneed = kneed;
        st->ties = kneed;
    }
}

// The first pass: the whole range.  BITS (of the later passes) 15: the next pass picks the bin; otherwise the last workgroup.
template <int BITS>
__global__ __launch_bounds__(kPassThreads) void osci_first_kernel(const float *W, int64_t nchunks, SelState *st, uint32_t *hist, uint32_t k_total)
{
    __shared__ float inv_tab[128], inv_bins[8];
    __shared__ uint32_t bins[kFirstBins];
    __shared__ uint32_t red[kPassWaves], flag;
    __shared__ uint2 picked;
    fill_inv_table(inv_tab);
    fill_inv_bins(inv_bins);
    for (int b = threadIdx.x; b < kFirstBins; b += kPassThreads) bins[b] = 0;
    __syncthreads();
    constexpr uint32_t kLow = (kFirstBin << 15) + 0x4000u;              // some pattern of bin 0, far from its ends
    const int64_t stride = (int64_t)gridDim.x * kPassThreads;          // a multiple of 16: rows of 16 lanes stay whole
    int64_t c = (int64_t)blockIdx.x * kPassThreads + threadIdx.x;
    F8 next{};
    if (c < nchunks) next = load8(W + c * 8);
    for (; c < nchunks; c += stride) {
        const F8 w = next;
        next = load8(W + (c + stride < nchunks ? c + stride : c) * 8);   // in flight while this chunk is counted
        Scores8 s = scores8(w, inv_tab, inv_bins);
        uint32_t nearest = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s.p[i] = s.p[i] > kLow ? s.p[i] : kLow;
            const uint32_t d = (s.p[i] + kNear) & 0x7FFFu;
            nearest = nearest < d ? nearest : d;
        }
        if (!s.ok || nearest <= 2 * kNear) {
#pragma unroll
            for (int i = 0; i < 8; ++i) s.p[i] = exact_score(s, i);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) atomicAdd(&bins[first_bin(s.p[i])], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kFirstBins; b += kPassThreads)
        if (bins[b]) atomicAdd(&hist[b], bins[b]);
    if (BITS == kBits || !last_to_arrive(&st->done[0], &flag)) return;
    const uint2 bin = pick_from_memory<kFirstBins>(hist, bins, red, &picked, k_total);
    store_interval(st, first_interval(bin.x), bin.y);
}

// A later pass, in 2^BITS bins.  With 15 bits PASS 1 takes the bin that every workgroup picks from the first pass's counts while its
// first weights are on their way (by the last workgroup of the first pass the choice took 2.5 us); otherwise the interval is
// that of the state.
constexpr int kAside = 2048;                               // elements put aside for an exact quotient
constexpr int later_lds(int bits) { return (4 << bits) + kAside * 8; }
template <int PASS, int BITS>
__global__ __launch_bounds__(kPassThreads) void osci_later_kernel(const float *W, int64_t nchunks, SelState *st, const uint32_t *first, uint32_t *hist, uint32_t k_total)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t bins[];
    constexpr int BINS = 1 << BITS;
    float2 *aside = reinterpret_cast<float2 *>(bins + BINS);
    __shared__ float inv_tab[128], inv_bins[8];
    __shared__ uint32_t red[kPassWaves], flag, n_aside;
    __shared__ uint2 picked;
    const int64_t stride = (int64_t)gridDim.x * kPassThreads;
    int64_t c = (int64_t)blockIdx.x * kPassThreads + threadIdx.x;
    F8 next{};
    SelInterval iv;
    uint32_t kneed;
    if (PASS == 1 && BITS == kBits) {
        if (c < nchunks) next = load8(W + c * 8);
        for (int b = threadIdx.x; b < kFirstBins; b += kPassThreads) bins[b] = first[b];
        __syncthreads();
        const uint2 bin = pick_bin<kFirstBins>(bins, red, &picked, k_total);
        iv = first_interval(bin.x);
        kneed = bin.y;
    } else {
        iv = st->iv;
        if (iv.width == 0) return;                         // uniform: the threshold is known
        kneed = st->kneed;
        if (c < nchunks) next = load8(W + c * 8);
    }
    const uint32_t within = reach(iv);
    fill_inv_table(inv_tab);
    fill_inv_bins(inv_bins);
    for (int b = threadIdx.x; b < BINS / 4; b += kPassThreads) reinterpret_cast<uint4 *>(bins)[b] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x == 0) n_aside = 0;
    __syncthreads();
    auto count = [&](uint32_t b) {
        if (b - iv.lo < within) atomicAdd(&bins[later_bin(iv, score_key(b), BITS)], 1u);
    };
    for (; c < nchunks; c += stride) {
        const F8 w = next;
        next = load8(W + (c + stride < nchunks ? c + stride : c) * 8);
        const Scores8 s = scores8(w, inv_tab, inv_bins);
        if (s.ok) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (s.p[i] - (iv.lo - kNear) <= within + 2 * kNear) {
                    const float width = bin_width(s.codes, i, s.unit);
                    const uint32_t a = atomicAdd(&n_aside, 1u);
                    if (a < kAside) aside[a] = make_float2(s.num.v[i], width);
                    else count(score_bits(s.num.v[i], width));
                }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) count(exact_score(s, i));
        }
    }
    __syncthreads();
    const uint32_t n = n_aside < kAside ? n_aside : kAside;
    for (uint32_t a = threadIdx.x; a < n; a += kPassThreads) count(score_bits(aside[a].x, aside[a].y));
    __syncthreads();
    for (int b = threadIdx.x; b < BINS; b += kPassThreads)
        if (bins[b]) atomicAdd(&hist[b], bins[b]);
    if (!last_to_arrive(&st->done[PASS], &flag)) return;
    const uint2 bin = pick_from_memory<BINS>(hist, bins, red, &picked, kneed);
    store_interval(st, next_interval(iv, bin.x, BITS), bin.y);
}

// flags of the lane's 8 elements against the threshold's key: bit i of gt / eq
__device__ __forceinline__ void score_flags(const Scores8 &s, uint32_t thr, uint32_t &gt, uint32_t &eq)
{
    uint32_t below = 0, nearest = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        const uint32_t d = s.p[i] - (thr - kNear);
        nearest = nearest < d ? nearest : d;
        below = (below << 1) | (d >> 31);                  // both lie below 2^31
    }
    gt = ~below & 0xFFu;
    eq = 0;
    if (!s.ok || nearest <= 2 * kNear) {
        const uint32_t last = last_pattern(thr);
        uint32_t ge = 0;
        gt = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t b = exact_score(s, i);
            gt |= (b > last ? 1u : 0u) << i;
            ge |= (b >= thr ? 1u : 0u) << i;
        }
        eq = ge ^ gt;
    }
}

// (greater, equal) counts per tile; the last workgroup replaces them by their exclusive prefix sums.  A workgroup takes
// four tiles at a time, four waves each.
__global__ __launch_bounds__(kPassThreads) void osci_count_kernel(const float *W, int64_t nchunks, SelState *st, uint32_t *counts, int64_t ntiles)
{
    __shared__ float inv_tab[128], inv_bins[8];
    __shared__ uint32_t red[2][kPassWaves], flag;
    fill_inv_table(inv_tab);
    fill_inv_bins(inv_bins);
    __syncthreads();
    const uint32_t thr = st->thr;
    const int64_t stride = (int64_t)gridDim.x * kPassThreads;
    const int64_t c0 = (int64_t)blockIdx.x * kPassThreads;
    F8 next{};
    if (c0 + threadIdx.x < nchunks) next = load8(W + (c0 + threadIdx.x) * 8);
    int set = 0;
    for (int64_t cb = c0; cb < nchunks; cb += stride, set ^= 1) {          // uniform over the workgroup
        const int64_t c = cb + threadIdx.x;
        const F8 w = next;
        if (c + stride < nchunks) next = load8(W + (c + stride) * 8);
        uint32_t gt = 0, eq = 0;
        if (c < nchunks) score_flags(scores8(w, inv_tab, inv_bins), thr, gt, eq);
        // both counts fit 16 bits (2048 elements per tile)
        uint32_t n = (uint32_t)__builtin_popcount(gt) | ((uint32_t)__builtin_popcount(eq) << 16);
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
        uint32_t *r = red[set];                            // two sets: one barrier per round
        if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = n;
        __syncthreads();
        const int64_t t = cb / kThreads + threadIdx.x;
        if (threadIdx.x < kPassThreads / kThreads && t < ntiles) {
            const uint32_t *q = r + 4 * threadIdx.x;
            const uint32_t sum = q[0] + q[1] + q[2] + q[3];
            store_dev(&counts[2 * t], sum & 0xFFFFu);
            store_dev(&counts[2 * t + 1], sum >> 16);
        }
    }
    if (!last_to_arrive(&st->done[4], &flag)) return;
    constexpr int kPer = 4;                                // tiles per thread and round
    uint32_t base_g = 0, base_e = 0;
    for (int64_t t0 = 0; t0 < ntiles; t0 += kPer * kPassThreads) {
        uint32_t vg[kPer], ve[kPer], sg = 0, se = 0, tot_g, tot_e;
        const int64_t t = t0 + (int64_t)threadIdx.x * kPer;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            vg[i] = t + i < ntiles ? load_dev(&counts[2 * (t + i)]) : 0u;
            ve[i] = t + i < ntiles ? load_dev(&counts[2 * (t + i) + 1]) : 0u;
            sg += vg[i];
            se += ve[i];
        }
        uint32_t pg = base_g + block_exclusive_scan<kPassWaves>(sg, red[0], tot_g);
        uint32_t pe = base_e + block_exclusive_scan<kPassWaves>(se, red[0], tot_e);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (t + i < ntiles) {
                counts[2 * (t + i)] = pg;
                counts[2 * (t + i) + 1] = pe;
            }
            pg += vg[i];
            pe += ve[i];
        }
        base_g += tot_g;
        base_e += tot_e;
    }
}

__global__ __launch_bounds__(kThreads) void osci_emit_kernel(const float *W, int64_t nchunks, const SelState *st, const uint32_t *offs,
                                                             uint32_t *idx, float *wp, float *qp, float *dm, float *dq, uint32_t k)
{
    __shared__ float inv_tab[128], inv_bins[8];
    __shared__ uint32_t red[4];
    fill_inv_table(inv_tab);
    fill_inv_bins(inv_bins);
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint32_t thr = st->thr, ties = st->ties;
    F8 w{{0, 0, 0, 0, 0, 0, 0, 0}}, q = w;
    uint32_t gt = 0, eq = 0;
    if (c < nchunks) {
        w = load8(W + c * 8);
        const Scores8 s = scores8(w, inv_tab, inv_bins);
        q = s.q;
        score_flags(s, thr, gt, eq);
    }
    // equal elements are ranked in index order over the whole tensor; the first `ties` of them are selected
    const uint32_t eq_tiles = offs[2 * blockIdx.x + 1], gt_tiles = offs[2 * blockIdx.x];
    uint32_t total;
    const uint32_t eq_before = eq_tiles + block_exclusive_scan<4>(__builtin_popcount(eq), red, total);
    uint32_t sel = gt, rank = eq_before;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((eq >> i) & 1u) {
            if (rank < ties) sel |= 1u << i;
            ++rank;
        }
    const uint32_t taken_eq_tiles = eq_tiles < ties ? eq_tiles : ties;       // selected equal elements of earlier tiles
    uint32_t pos = gt_tiles + taken_eq_tiles + block_exclusive_scan<4>(__builtin_popcount(sel), red, total);
    if (pos + __builtin_popcount(sel) > k) sel = 0;        // k are selected: this only keeps the stores inside the arrays
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((sel >> i) & 1u) {
            idx[pos] = (uint32_t)(c * 8 + i);
            wp[pos] = w.v[i];
            qp[pos] = q.v[i];
            dm[pos] = 0.0f;
            dq[pos] = 0.0f;
            ++pos;
        }
}

// First position j in the ascending list idx[0..k) with idx[j] >= e, by one whole wave: 64 probes per step, so that a
// list of 400 000 entries takes four dependent loads instead of nineteen.
__device__ __forceinline__ int64_t wave_lower_bound(const uint32_t *idx, int64_t k, int64_t e)
{
    const int lane = threadIdx.x & 63;
    int64_t lo = 0, n = k;                                 // the answer is in [lo, lo + n]
    while (n > 0) {
        const int64_t step = (n + 63) / 64;
        const int64_t j = lo + step * (lane + 1) - 1;      // the last entry of the lane's piece
        const bool below = j < lo + n && (int64_t)idx[j] < e;
        const int pieces = __builtin_popcountll(__ballot(below));
        const int64_t left = n - step * pieces;
        lo += step * pieces;
        // every piece that ends below e is behind us; the answer lies in the next one (its last entry is not below e, or
        // it is the unfinished piece at the end)
        n = left <= 0 ? 0 : (step - 1 < left ? step - 1 : left);
        if (step == 1) break;
    }
    return lo;
}

// Alg. 3 at a later step (SUPPRESS = false) and Alg. 1 on the tracked subset (SUPPRESS = true).  A workgroup takes T tiles
// of 2048 consecutive weights: Q of the tiles goes to LDS, then their entries of the (ascending) index list are updated
// from it.  The call is bound by its chain of dependent loads (search, entries, weights), so the weights are fetched
// before the search (`dense`: lists in which nearly every tile has entries; otherwise tiles without a tracked weight stop
// after the search and read nothing else), and a long tensor takes several tiles per search: 8192 x 1024 with 5 % tracked
// took 21 us with one tile and a one-thread search, 14 us like this.
template <bool SUPPRESS, int T>
__global__ __launch_bounds__(kThreads) void osci_sparse_kernel(float *W, int64_t nchunks, const uint32_t *idx, int64_t k, float *wp,
                                                               float *qp, float *dm, float *dq, float tau,
                                                               unsigned long long *n_reset, int dense)
{
    __shared__ float inv_tab[128];
    __shared__ __attribute__((aligned(16))) float qt[T * kTile];
    __shared__ int64_t range[2];
    __shared__ unsigned int wg_count;
    const int64_t tile0 = (int64_t)blockIdx.x * (T * kTile);
    const int64_t c0 = (int64_t)blockIdx.x * (T * kThreads) + threadIdx.x;
    F8 w[T];
    auto fetch = [&]() {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int64_t c = c0 + t * kThreads;
            w[t] = load8(W + (c < nchunks ? c : nchunks - 1 - ((nchunks - 1 - c) & 15)) * 8);   // past the end: some valid chunk, not used
        }
    };
    if (dense) fetch();
    fill_inv_table(inv_tab);
    const int wave = threadIdx.x >> 6;
    if (wave < 2) {
        const int64_t j = wave_lower_bound(idx, k, tile0 + wave * (T * kTile));
        if ((threadIdx.x & 63) == 0) range[wave] = j;
    }
    if (threadIdx.x == 0) wg_count = 0;
    __syncthreads();
    const int64_t j0 = range[0], j1 = range[1];
    if (j0 == j1) return;                                  // uniform
    if (!dense) fetch();
#pragma unroll
    for (int t = 0; t < T; ++t)
        if (c0 + t * kThreads < nchunks) store8(qt + (t * kThreads + threadIdx.x) * 8, quant_dequant8(w[t], inv_tab));
    __syncthreads();                                       // every weight of the tiles has been read: resets may follow
    unsigned int mine = 0;
    // Four entries per thread and step, their loads in flight together: a list whose entries lie close together (equal scores
    // are taken in index order) leaves a workgroup with up to T * 2048 of them, and one per step was a chain of 8 T round trips
    // (8192 x 1024 zeros, 5 % tracked, four tiles: 35 us, 16.5 like this).
    constexpr int kU = 4;
    for (int64_t jb = j0 + threadIdx.x; jb < j1; jb += kU * kThreads) {
        uint32_t e[kU];
        float m[kU], d[kU], p[kU], r[kU], wv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t j = jb + u * kThreads;
            if (j >= j1) break;
            e[u] = idx[j];
            m[u] = dm[j];
            d[u] = dq[j];
            if (!SUPPRESS) {
                p[u] = wp[j];
                r[u] = qp[j];
            }
        }
        if (!SUPPRESS) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (jb + u * kThreads >= j1) break;
                wv[u] = W[e[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t j = jb + u * kThreads;
            if (j >= j1) break;
            const float q = qt[e[u] - tile0];
            if (SUPPRESS) {
                const float risk = d[u] / m[u];            // IEEE quotient; 0 / 0 is NaN and compares false
                if (risk >= tau) {
                    W[e[u]] = q;
                    ++mine;
                }
            } else {
                dm[j] = m[u] + fabsf(wv[u] - p[u]);
                dq[j] = d[u] + fabsf(q - r[u]);
                wp[j] = wv[u];
                qp[j] = q;
            }
        }
    }
    if (SUPPRESS && n_reset) {
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
        if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&wg_count, mine);
        __syncthreads();
        if (threadIdx.x == 0 && wg_count) atomicAdd(n_reset, (unsigned long long)wg_count);
    }
}

template <bool SUPPRESS>
hipError_t launch_sparse(float *W, int64_t n, const uint32_t *idx, int64_t k, float *wp, float *qp, float *dm, float *dq, float tau,
                         unsigned long long *n_reset, hipStream_t st)
{
    const int64_t nchunks = n / 8;
    if (nchunks == 0 || k == 0) return hipSuccess;
    const int64_t ntiles = (nchunks + kThreads - 1) / kThreads;
    const int dense = k >= ntiles;                         // on average at least one entry per tile
    // Several tiles per workgroup once that still leaves two workgroups per CU: four in the reset, whose workgroups each end
    // with an addition to one counter (8192 x 1024, resets all over the tensor: 59 us with one tile, 35 with two, 23 with
    // four).  The step has no counter: two, which keeps a list whose entries lie close together on twice the workgroups
    // (8192 x 1024 zeros, 5 % tracked: 11.6 us with one, 12.8 with two, 16.5 with four; spread evenly 15.6 / 13.5 / 13.1), and
    // four from 16384 tiles on (8192 x 8192, 5 %: 126 / 111 / 95; zeros 88 / 73 / 65).
    auto launch = [&](auto t) {
        constexpr int T = decltype(t)::value;
        hipLaunchKernelGGL((osci_sparse_kernel<SUPPRESS, T>), dim3((unsigned)((ntiles + T - 1) / T)), dim3(kThreads), 0, st, W, nchunks, idx, k,
                           wp, qp, dm, dq, tau, n_reset, dense);
    };
    if (ntiles < 2048) launch(std::integral_constant<int, 1>{});
    else if (!SUPPRESS && ntiles < 16384) launch(std::integral_constant<int, SUPPRESS ? 4 : 2>{});
    else launch(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

}  // namespace

size_t osci_select_workspace_bytes(int64_t n)
{
    const int64_t ntiles = (n + kTile - 1) / kTile;
    return 256 + kFirstBins * sizeof(uint32_t) + (size_t)ntiles * 2 * sizeof(uint32_t);
}

hipError_t launch_osci_select(const float *W, int64_t n, int64_t k, uint32_t *idx, float *wp, float *qp, float *dm, float *dq,
                              void *ws, hipStream_t st)
{
    const int64_t nchunks = n / 8;
    if (nchunks == 0 || k == 0) return hipSuccess;
    static const hipError_t attr = []() {                  // once; the initialisation of a function-local static is thread-safe
        for (auto kern : {osci_later_kernel<1, kBits>, osci_later_kernel<2, kBits>}) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, later_lds(kBits));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return attr;
    SelState *state = static_cast<SelState *>(ws);
    uint32_t *hist = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(ws) + 256);
    uint32_t *counts = hist + kFirstBins;
    const int64_t ntiles = (nchunks + kThreads - 1) / kThreads;
    const int64_t want = (nchunks + kPassThreads - 1) / kPassThreads;
    const dim3 grid((unsigned)(want < kPassWgs ? want : kPassWgs)), block(kPassThreads);
    // The counts of the 32768 bins take the place of the indices, which are written last; fewer indices than bins: 2048 bins in
    // the workspace, and one pass more (256 x 256, 5 %: a launch-bound call either way).
    if (k >= kBins) {
        hipLaunchKernelGGL(osci_zero_kernel, dim3((kFirstBins + kBins) / kThreads), dim3(kThreads), 0, st, state, hist, idx);
        hipLaunchKernelGGL(osci_first_kernel<kBits>, grid, block, 0, st, W, nchunks, state, hist, (uint32_t)k);
        hipLaunchKernelGGL((osci_later_kernel<1, kBits>), grid, block, later_lds(kBits), st, W, nchunks, state, hist, idx, (uint32_t)k);
        hipLaunchKernelGGL((osci_later_kernel<2, kBits>), grid, block, later_lds(kBits), st, W, nchunks, state, hist, idx, (uint32_t)k);
    } else {
        hipLaunchKernelGGL(osci_zero_kernel, dim3(kFirstBins / kThreads), dim3(kThreads), 0, st, state, hist, nullptr);
        hipLaunchKernelGGL(osci_first_kernel<kFewBits>, grid, block, 0, st, W, nchunks, state, hist, (uint32_t)k);
        hipLaunchKernelGGL((osci_later_kernel<1, kFewBits>), grid, block, later_lds(kFewBits), st, W, nchunks, state, nullptr, hist, (uint32_t)k);
        hipLaunchKernelGGL((osci_later_kernel<2, kFewBits>), grid, block, later_lds(kFewBits), st, W, nchunks, state, nullptr, hist, (uint32_t)k);
        hipLaunchKernelGGL((osci_later_kernel<3, kFewBits>), grid, block, later_lds(kFewBits), st, W, nchunks, state, nullptr, hist, (uint32_t)k);
    }
    hipLaunchKernelGGL(osci_count_kernel, grid, block, 0, st, W, nchunks, state, counts, ntiles);
    hipLaunchKernelGGL(osci_emit_kernel, dim3((unsigned)ntiles), dim3(kThreads), 0, st, W, nchunks, state, counts, idx, wp, qp, dm, dq,
                       (uint32_t)k);
    return hipGetLastError();
}

hipError_t launch_osci_update_sparse(const float *W, int64_t n, const uint32_t *idx, int64_t k, float *wp, float *qp, float *dm,
                                     float *dq, hipStream_t st)
{
    return launch_sparse<false>(const_cast<float *>(W), n, idx, k, wp, qp, dm, dq, 0.0f, nullptr, st);
}

hipError_t launch_osci_suppress_sparse(float *W, int64_t n, const uint32_t *idx, int64_t k, const float *dm, const float *dq,
                                       float tau, unsigned long long *n_reset, hipStream_t st)
{
    return launch_sparse<true>(W, n, idx, k, nullptr, nullptr, const_cast<float *>(dm), const_cast<float *>(dq), tau, n_reset, st);
}

hipError_t launch_osci_update(const float *W, float *W_prev, float *dist_m, float *dist_q, int64_t n, int first, hipStream_t st)
{
    const int64_t nchunks = n / 8;
    if (nchunks == 0) return hipSuccess;
    const unsigned grid = (unsigned)((nchunks + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(osci_update_kernel, dim3(grid), dim3(kThreads), 0, st, W, W_prev, dist_m, dist_q, nchunks, first);
    return hipGetLastError();
}

hipError_t launch_osci_suppress(float *W, const float *dist_m, const float *dist_q, float tau, int64_t n,
                                unsigned long long *n_reset, hipStream_t st)
{
    const int64_t nchunks = n / 8;
    if (nchunks == 0) return hipSuccess;
    const int64_t want = (nchunks + kThreads - 1) / kThreads;
    const unsigned grid = (unsigned)(!n_reset || want < kMaxCountingWgs ? want : kMaxCountingWgs);
    hipLaunchKernelGGL(osci_suppress_kernel, dim3(grid), dim3(kThreads), 0, st, W, dist_m, dist_q, tau, nchunks, n_reset);
    return hipGetLastError();
}

}  // namespace tj
