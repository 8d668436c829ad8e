"""The search for the k-th largest sensitivity score on the CPU: the key and interval functions the selection kernels use
(csrc/osci_search.h), run through the same passes by a host program, select exactly k elements - equal scores in ascending
index order, NaN above infinity - whatever the scores are."""
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
static bool pick(const long *hist, long &kneed, uint32_t &bin)
{
    long above = 0;
    for (int b = kBins - 1; b >= 0; --b) {
        if (above < kneed && kneed <= above + hist[b]) { bin = (uint32_t)b; kneed -= above; return true; }
        above += hist[b];
    }
    return false;
}

// sel[i] = 1 for the selected elements; returns their number, or -1 - pass where a pass found no bin
extern "C" long select_k(const uint32_t *score, long n, long k, unsigned char *sel)
{
    SelInterval iv{};
    long kneed = k;
    for (int pass = 0; pass < 4; ++pass) {
        if (pass > 0 && iv.width == 0) break;
        long hist[kBins] = {};
        for (long i = 0; i < n; ++i) {
            if (pass == 0) ++hist[first_bin(score[i])];
            else if (score[i] - iv.lo < reach(iv)) {
                const uint32_t key = reach(iv) != iv.span ? score_key(score[i]) : score[i];    // the kernel's two loops
                if (later_bin(iv, key) >= (uint32_t)kBins) return -20 - pass;
                ++hist[later_bin(iv, key)];
            }
        }
        uint32_t bin = 0;
        if (!pick(hist, kneed, bin)) return -1 - pass;
        iv = pass == 0 ? first_interval(bin) : next_interval(iv, bin);
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
"""


@pytest.fixture(scope="module")
def select(tmp_path_factory):
    d = tmp_path_factory.mktemp("osci_search")
    src, lib = d / "harness.cpp", d / "libharness.so"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2510_27527_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    fn = C.CDLL(str(lib)).select_k
    fn.restype = C.c_long
    fn.argtypes = [C.c_void_p, C.c_long, C.c_long, C.c_void_p]

    def run(score, k):
        bits = np.ascontiguousarray(score).view(np.uint32)
        sel = np.zeros(bits.size, np.uint8)
        return fn(bits.ctypes.data, bits.size, k, sel.ctypes.data), np.flatnonzero(sel)
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
