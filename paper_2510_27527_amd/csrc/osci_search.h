// Search for the k-th largest sensitivity score (osci.hip): how a score becomes a key, and how each histogram pass narrows
// the interval of keys that holds the threshold.  Plain constexpr functions, so that the kernels and a host program run the
// same code.
#pragma once
#include <stdint.h>

namespace tj {

// Scores are non-negative, so they order like their binary32 patterns.  A NaN (the score of a NaN weight, and of the whole
// outer block of an infinite one) ranks above infinity: all of its patterns, of either sign, share one key, so that every pass
// counts exactly the elements that the passes before it counted.  The passes test the raw pattern against bounds that take
// the NaNs in; only a pattern inside the interval is turned into its key.
constexpr uint32_t kNaNKey = 0x7F800001u;
constexpr uint32_t score_key(uint32_t pattern) { return pattern < kNaNKey ? pattern : kNaNKey; }
constexpr uint32_t last_pattern(uint32_t key) { return key == kNaNKey ? 0xFFFFFFFFu : key; }   // the largest pattern of the key

constexpr int kFirstBins = 2048, kBits = 15, kBins = 1 << kBits;       // bins of the first pass and of a later one
constexpr int kFewBits = 11;                                           // of a later one where memory for kBins is not at hand
// The first pass: 256 bins per octave in [2^-8, 1] (the last of them holds 1 itself), an open bin below and one above.
constexpr uint32_t kFirstBin = (0x3F800000u >> 15) - (kFirstBins - 2);   // pattern >> 15 of bin 0; 1.0 falls into bin 2046
constexpr int first_bin(uint32_t pattern)
{
    const int d = (int)(pattern >> 15) - (int)kFirstBin;
    return d < 0 ? 0 : d > kFirstBins - 1 ? kFirstBins - 1 : d;
}

struct SelInterval {
    uint32_t lo, span;    // [lo, lo + span) holds the threshold; every key of the bin it came from lies inside
    uint32_t width;       // bits still open: span <= 2^width
};
constexpr SelInterval first_interval(uint32_t bin)
{
    if (bin == 0) return {0u, (kFirstBin + 1) << 15, 30u};
    const uint32_t lo = (kFirstBin + bin) << 15;
    if (bin == kFirstBins - 1) return {lo, 1u << 30, 30u};
    return {lo, 1u << 15, 15u};
}
static_assert(first_interval(kFirstBins - 1).lo + (1u << 30) > kNaNKey, "the open top bin ends above the largest key");
static_assert((((kFirstBin + 1) << 15) >> 30) == 0, "the open bottom bin fits its width");

// a later pass: 2^bits bins of 2^shift keys (15 bits: 30 -> 15 -> 0 open bits, 15 -> 0; 11 bits: 30 -> 19 -> 8 -> 0, 15 -> 4 -> 0)
constexpr uint32_t later_shift(uint32_t width, int bits = kBits) { return width > (uint32_t)bits ? width - bits : 0; }
// a pattern belongs to the interval if pattern - lo < reach (unsigned: patterns below lo wrap around)
constexpr uint32_t reach(const SelInterval &s) { return kNaNKey - s.lo < s.span ? 0u - s.lo : s.span; }
constexpr uint32_t later_bin(const SelInterval &s, uint32_t key, int bits = kBits) { return (key - s.lo) >> later_shift(s.width, bits); }
constexpr SelInterval next_interval(const SelInterval &s, uint32_t bin, int bits = kBits)
{
    const uint32_t shift = later_shift(s.width, bits), left = s.span - (bin << shift);
    return {s.lo + (bin << shift), left < (1u << shift) ? left : 1u << shift, shift};
}

// An estimate further than this many patterns from a value is on the same side of it as the exact score (osci.hip has the bound).
constexpr uint32_t kNear = 16;

}  // namespace tj
