"""The search for the k-th largest sensitivity score on the CPU: the key and interval functions the selection kernels use
(csrc/osci_search.h), run through the same passes by a host program, select exactly k elements - equal scores in ascending
index order, NaN above infinity - whatever the scores are, with the bins of either kind of later pass; and the margin around an
estimated score covers its error."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "osci_search.h"
using namespace tj;

// the bin, counted from the top, that holds the kneed-th key; false if there is none
static bool pick(const long *hist, int bins, long &kneed, uint32_t &bin)
{
    long above = 0;
    for (int b = bins - 1; b >= 0; --b) {
        if (above < kneed && kneed <= above + hist[b]) { bin = (uint32_t)b; kneed -= above; return true; }
        above += hist[b];
    }
    return false;
}

extern "C" int bits_of(int few) { return few ? kFewBits : kBits; }

// sel[i] = 1 for the selected elements; returns their number, or -1 - pass where a pass found no bin.  Later passes have 2^bits
// bins: two of them with 15 bits, three with 11.
extern "C" long select_k(const uint32_t *score, long n, long k, unsigned char *sel, int bits)
{
    SelInterval iv{};
    long kneed = k;
    static long hist[kBins];
    for (int pass = 0; pass < (bits == kBits ? 3 : 4); ++pass) {
        if (pass > 0 && iv.width == 0) break;
        const int bins = pass == 0 ? kFirstBins : 1 << bits;
        for (int b = 0; b < bins; ++b) hist[b] = 0;
        for (long i = 0; i < n; ++i) {
            if (pass == 0) ++hist[first_bin(score[i])];
            else if (score[i] - iv.lo < reach(iv)) {
                const uint32_t b = later_bin(iv, score_key(score[i]), bits);
                if (b >= (uint32_t)bins) return -20 - pass;
                ++hist[b];
            }
        }
        uint32_t bin = 0;
        if (!pick(hist, bins, kneed, bin)) return -1 - pass;
        iv = pass == 0 ? first_interval(bin) : next_interval(iv, bin, bits);
    }
    if (iv.width != 0) return -9;
    long total = 0, ties = 0;
    for (long i = 0; i < n; ++i) {
        const bool gt = score[i] > last_pattern(iv.lo), eq = score[i] >= iv.lo && !gt;
        sel[i] = gt || (eq && ties++ < kneed);
        total += sel[i];
    }
    return total;
}

static uint32_t f2u(float f) { uint32_t u; __builtin_memcpy(&u, &f, 4); return u; }
static float u2f(uint32_t u) { float f; __builtin_memcpy(&f, &u, 4); return f; }

extern "C" int margin() { return (int)kNear; }

// Largest difference in patterns between the estimate |x - Q(x)| * (1 / unit) * (1 / bin), its reciprocal `off` patterns from the rounded one
// (the hardware's is within one), and the exact quotient, over n pairs and all bin lengths.
extern "C" long estimate_error(const float *num, const float *unit, long n, int off)
{
    const float bins[4] = {0.5f, 0.75f, 1.0f, 1.5f}, inv[4] = {2.0f, 4.0f / 3.0f, 1.0f, 2.0f / 3.0f};
    long worst = 0;
    for (long i = 0; i < n; ++i) {
        const float y = u2f(f2u(1.0f / unit[i]) + (uint32_t)off);
        for (int b = 0; b < 4; ++b) {
            const long e = (long)f2u(num[i] * y * inv[b]) - (long)f2u(num[i] / (bins[b] * unit[i]));
            if (e > worst || -e > worst) worst = e < 0 ? -e : e;
        }
    }
    return worst;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("osci_search")
    src, lib = d / "harness.cpp", d / "libharness.so"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2510_27527_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


@pytest.fixture(scope="module", params=["32768 bins", "2048 bins"])
def select(harness, request):
    fn = harness.select_k
    fn.restype = C.c_long
    fn.argtypes = [C.c_void_p, C.c_long, C.c_long, C.c_void_p, C.c_int]
    width = harness.bits_of(request.param == "2048 bins")
    assert 1 << width == int(request.param.split()[0])

    def run(score, k):
        bits = np.ascontiguousarray(score).view(np.uint32)
        sel = np.zeros(bits.size, np.uint8)
        return fn(bits.ctypes.data, bits.size, k, sel.ctypes.data, width), np.flatnonzero(sel)
    return run


def expected(score, k):
    """the k largest, NaN above everything, ties in index order"""
    key = np.full(score.size, np.inf)
    number = ~np.isnan(score)
    key[number] = np.minimum(score[number].astype(np.float64), 1e300)
    return np.sort(np.argsort(-key, kind="stable")[:k])


def score_sets():
    rng = np.random.default_rng(4)
    ordinary = rng.random(8192).astype(np.float32) ** 2
    nan = np.array([0x7FC00000, 0xFFC00000, 0x7F800001, 0xFFFFFFFF, 0x7FFFFFFF], np.uint32).view(np.float32)

    def planted(count, values):
        s = ordinary.copy()
        s[rng.choice(s.size, count, replace=False)] = rng.choice(values, count)
        return s
    return {"ordinary": ordinary, "zero": np.zeros(8192, np.float32), "one": np.ones(8192, np.float32),
            "ties": rng.choice(np.array([0, 1e-30, 0.25, 0.5, 1.0], np.float32), 8192),
            "tiny": (ordinary * np.float32(1e-38)), "huge": ordinary * np.float32(1e38),
            "one NaN": planted(1, nan), "512 NaN": planted(512, nan), "all NaN": np.resize(nan, 8192),
            "inf": planted(128, np.array([np.inf], np.float32)),
            "NaN and inf": planted(700, np.concatenate([nan, np.array([np.inf, 3e38], np.float32)]))}


@pytest.mark.parametrize("name", list(score_sets()))
def test_exactly_k_are_selected(select, name):
    s = score_sets()[name]
    nans = int(np.isnan(s).sum())
    for k in sorted({1, 64, 127, 128, 129, 410, 512, 4096, s.size - 1, s.size} | {max(1, nans - 1), max(1, nans), nans + 1} - {s.size + 1}):
        count, idx = select(s, k)
        assert count == k, (name, k)
        want = expected(s, k)
        assert np.array_equal(idx, want), (name, k)


def test_margin_covers_the_error_of_an_estimate(harness):
    """Units over the range in which the passes estimate, distances from the smallest subnormal to eight units.  The bound, in units of 2^-24
    relative, is 7 in all: reciprocal 2, two products 2, rounded 4/3 and 2/3 1, rounded bin length 1, quotient 1; at most 14 patterns,
    where the exact value lies just above a power of two."""
    fn = harness.estimate_error
    fn.restype = C.c_long
    fn.argtypes = [C.c_void_p, C.c_void_p, C.c_long, C.c_int]
    rng = np.random.default_rng(6)
    n = 1 << 18
    unit = np.ldexp(rng.uniform(1, 2, n), rng.integers(-99, 99, n)).astype(np.float32)
    sets = [unit * rng.uniform(0, 8, n).astype(np.float32),                        # ordinary distances
            unit * np.ldexp(rng.uniform(1, 2, n), rng.integers(-60, 3, n)).astype(np.float32),
            rng.integers(0, 1 << 20, n).astype(np.uint32).view(np.float32),           # subnormal distances
            unit * np.ldexp(1.0, rng.integers(-8, 1, n)).astype(np.float32)]          # scores next to powers of two
    worst = 0
    for num in sets:
        num = np.ascontiguousarray(num, dtype=np.float32)
        for off in (-1, 0, 1):
            worst = max(worst, fn(num.ctypes.data, unit.ctypes.data, n, off))
    assert 0 < worst <= 14 < harness.margin(), worst
