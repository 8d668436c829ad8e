"""The launchers refuse operands in a layout that the kernel they would start does not read or write: on the host, before anything is
launched, so a program without a GPU sees it (what is accepted ends here with the runtime's "no device" instead)."""
import ctypes as C
import itertools
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27527_amd", "csrc")
INVALID = 1                      # hipErrorInvalidValue

HARNESS = r"""
#include "internal.h"
using namespace tj;

static uint8_t *const kFar = reinterpret_cast<uint8_t *>(0x7F0000001000);      // never dereferenced

static GemmOperand operand(int64_t rows, int outer, int blocked) { return GemmOperand{kFar, kFar, reinterpret_cast<float *>(kFar), rows, outer, blocked}; }

extern "C" int product(int64_t M, int64_t N, int64_t K, int outer, int a_blocked, int b_blocked)
{
    return launch_gemm_nt(operand(M, outer, a_blocked), operand(N, outer, b_blocked), K, kFar, 0, kFar, (size_t)1 << 40, nullptr);
}

extern "C" int group(const int64_t *mnk, int n, int outer, const int *blocked)
{
    GemmProduct p[3];
    for (int i = 0; i < n; ++i)
        p[i] = GemmProduct{operand(mnk[3 * i], outer, blocked[i]), operand(mnk[3 * i + 1], outer, blocked[i]), mnk[3 * i + 2], kFar};
    return launch_gemm_group(plan_group(reinterpret_cast<const int64_t (*)[3]>(mnk), n, outer, false), p, 0, kFar, (size_t)1 << 40, nullptr);
}

// kind: 0 row-wise, 1 two row-wise ones, 2 column-wise, 3 both of one tensor, 4 column-wise from a packed one, 5 two of them, 6 and a maximum
extern "C" int quantize(int kind, int64_t R, int64_t C, int rounding, int scale_up, int outer, int blocked0, int blocked1)
{
    float *const f = reinterpret_cast<float *>(kFar);
    QuantParams p{};
    p.rounding = rounding;
    p.scale_up = scale_up;
    p.outer = outer;
    p.amax_scalar = f;
    const QuantOut o0{kFar, kFar, f, nullptr, blocked0}, o1{kFar, kFar, f, nullptr, blocked1};
    const PackedSrc s{kFar, kFar, f, outer};
    int npart = 0;
    switch (kind) {
        case 0: return launch_quant_row_bf16(kFar, R, C, p, o0, nullptr);
        case 1: return launch_quant_row_bf16_pair(kFar, R, C, p, o0, kFar, R, C, p, o1, nullptr);
        case 2: return launch_quant_col_bf16(kFar, R, C, p, o0, nullptr);
        case 3: return launch_quant_dual_bf16(kFar, R, C, p, o0, p, o1, nullptr);
        case 4: return launch_requant_col(s, R, C, p, o0, nullptr);
        case 5: return launch_requant_col_pair(s, R, C, p, o0, s, R, C, p, o1, nullptr);
        default: return launch_requant_col_pair_amax(s, R, C, p, o0, s, R, C, p, o1, kFar, R * C, f, &npart, nullptr);
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if torch.cuda.is_available():
        pytest.skip("made-up addresses: only where nothing can be launched")
    import paper_2510_27527_amd.binding as B
    from paper_2510_27527_amd import build
    B.lib()
    d = tmp_path_factory.mktemp("layouts")
    src, so = d / "harness.hip", d / "harness.so"
    src.write_text(HARNESS)
    where = os.path.dirname(B.LIB_PATH)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["-shared", "-I", CSRC, str(src), "-o", str(so), "-L" + where, "-ltjnvfp4",
                                                                                    "-Wl,-rpath," + where], check=True)
    return C.CDLL(str(so))


def _kernel(M, N, K, outer):
    import paper_2510_27527_amd.binding as B
    return B.gemm_splits_waves(M, N, K, outer), B.gemm_plan(M, N, K, outer)[2]


def _product(lib, M, N, K, outer, a, b):
    i64 = C.c_int64
    return lib.product(i64(M), i64(N), i64(K), outer, a, b)


def _group(lib, products, outer, blocked):
    flat = [v for p in products for v in p]
    return lib.group((C.c_int64 * len(flat))(*flat), len(products), outer, (C.c_int * len(blocked))(*blocked))


# (outer mode, M, N, K, whether the waves split the reduction, K splits, whether blocked operands can be read)
PRODUCTS = [(0, 2048, 2048, 320, False, 1, True), (0, 1024, 1024, 2048, True, 1, False), (0, 64, 64, 1088, False, 2, False), (0, 64, 64, 1024, False, 2, True),
            (1, 2048, 2048, 512, False, 1, True), (1, 2048, 2048, 384, False, 1, False), (1, 1024, 1024, 2048, True, 1, False),
            (1, 256, 128, 3328, False, 2, True)]


@pytest.mark.parametrize("outer,M,N,K,waves,split,takes", PRODUCTS)
def test_products_refuse_a_layout_they_do_not_read(lib, outer, M, N, K, waves, split, takes):
    got = _kernel(M, N, K, outer)
    assert got[0] == waves and (got[1] > 1) == (split > 1)
    assert _product(lib, M, N, K, outer, 0, 0) not in (0, INVALID)
    assert (_product(lib, M, N, K, outer, 1, 1) == INVALID) == (not takes)
    assert _product(lib, M, N, K, outer, 1, 0) == INVALID and _product(lib, M, N, K, outer, 0, 1) == INVALID


# (outer mode, N, D, H, C of a backward call: dX, dW and with H the outlier channels' dX, tile of the launch together, layouts accepted)
BACKWARD = [(0, 320, 4160, 0, 512, (128, 128), {(0, 0), (1, 1)}), (0, 320, 128, 0, 256, (64, 64), {(0, 0)}),
            (1, 512, 6272, 0, 512, (256, 128), {(0, 0), (1, 1)}), (1, 896, 3328, 0, 3456, (128, 128), {(0, 0)}),
            (0, 8192, 768, 0, 3072, (0, 0), {(0, 0), (1, 0)}), (1, 5504, 1024, 0, 256, (0, 0), {(0, 0), (1, 0)}),
            (0, 256, 6528, 640, 256, (128, 128), {(0, 0, 0), (1, 1, 1)}), (1, 256, 384, 32, 256, (64, 64), {(0, 0, 0), (1, 1, 1)})]


@pytest.mark.parametrize("outer,N,D,H,Cc,tile,accepted", BACKWARD)
def test_launches_of_several_products_refuse_layouts_they_do_not_read(lib, outer, N, D, H, Cc, tile, accepted):
    import paper_2510_27527_amd.binding as B
    assert B.backward_plan(N, D, H, Cc, outer) == tile
    products = [(N, D, Cc), (Cc, D, N)] + ([(N, H, Cc)] if H else [])
    for blocked in itertools.product((0, 1), repeat=len(products)):
        assert (_group(lib, products, outer, blocked) != INVALID) == (blocked in accepted), blocked


@pytest.mark.parametrize("rounding,scale_up", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("kind", range(7))
def test_quantizers_refuse_a_layout_they_do_not_write(lib, kind, rounding, scale_up):
    def quantize(R, Cc, outer, b0, b1):
        return lib.quantize(kind, C.c_int64(R), C.c_int64(Cc), rounding, scale_up, outer, b0, b1) != INVALID
    backward = rounding == 1 and scale_up == 1
    for outer in (0,) if kind == 3 else (0, 1):
        assert quantize(256, 256, outer, 0, 0)
        for b0, b1 in ((1, 1), (1, 0), (0, 1)):
            second = kind in (1, 3, 5, 6)
            if not second and not b0:
                continue
            # the row-wise pair is the forward call's; column-wise kernels write blocked operands of every rounding
            assert quantize(256, 256, outer, b0, b1) == (kind != 1 and (kind not in (0, 3) or backward)), (outer, b0, b1)
            # a row of the output is no whole number of 64s
            if outer == 0:
                axis_c = (b0 and kind in (0, 1, 3)), (b1 and kind == 1)
                axis_r = (b0 and kind in (2, 4, 5, 6)), (b1 and kind in (3, 5, 6))
                assert not quantize(256 + 32 * any(axis_r), 256 + 32 * any(axis_c), outer, b0, b1), (b0, b1)
    rows, cols = ((1 << 24) + 64, 64) if kind < 2 else (128, (1 << 24) + 64)
    assert not quantize(rows, cols, 0, *((0, 1) if kind == 3 else (1, 1)))
