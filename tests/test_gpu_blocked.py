"""The backward quantizers write their operands blocked along K for the products (codes [K/64][rows][32 bytes], scale bytes
[ceil(K/256)][rows][16], outer scales [K/128][rows]).  The layout changes no value, so the gradients have to be, byte for byte, the products of
the row-major operands that the public quantizer calls write, which are compared with the oracle elsewhere."""
import math
import random

import pytest

torch = pytest.importorskip("torch")

# (outer mode, transform, N, D, C): reductions N and C of 0, 64, 128 and 192 mod 256, in one piece and split (split on an odd number of 64s: row-major),
# outputs that end inside a tile, row-wise tiles of 256 and 512 columns
CASES = [
    (0, 0, 64, 64, 64), (0, 0, 192, 128, 128), (0, 0, 128, 64, 192), (0, 0, 256, 64, 256), (0, 0, 1024, 64, 64), (0, 0, 64, 64, 1088),
    (0, 0, 1152, 64, 64), (0, 0, 64, 80, 1216), (0, 0, 640, 1664, 256), (0, 0, 512, 3520, 576), (0, 0, 2112, 3776, 64), (0, 0, 64, 2496, 3200),
    (0, 0, 192, 3648, 1088), (0, 0, 3840, 1600, 256), (0, 0, 128, 4544, 2816), (0, 0, 1600, 1216, 512), (0, 0, 3520, 3520, 128), (0, 0, 4096, 768, 3072),
    (1, 0, 256, 256, 256), (1, 1, 2048, 256, 256), (1, 0, 256, 4224, 256), (1, 1, 256, 128, 1024), (1, 0, 256, 1280, 3328), (1, 1, 3328, 1792, 256),
    (1, 0, 256, 4096, 1536), (1, 1, 384, 256, 512), (1, 0, 512, 256, 640),
]
# with the ones above: every instantiation of the product kernel that reads blocked operands, by tile, scale fetch, alone, split or together
REACH = [
    (0, 0, 256, 4560, 256), (0, 0, 256, 4320, 320), (0, 0, 2560, 144, 1152), (0, 0, 6656, 16, 4992), (0, 0, 7168, 16, 3136), (0, 0, 320, 6624, 256),
    (0, 0, 256, 5632, 512), (0, 0, 512, 8128, 256), (0, 0, 320, 6928, 576), (0, 0, 64, 5424, 4672), (0, 0, 256, 5680, 1344), (0, 0, 5632, 8176, 64),
    (0, 0, 7616, 1568, 256), (0, 0, 1280, 6640, 768), (0, 0, 8960, 464, 5696),
    (1, 0, 256, 2176, 256), (1, 1, 256, 5504, 512), (1, 0, 256, 8192, 512), (1, 1, 2816, 384, 5888), (1, 0, 9472, 256, 2432),
    (0, 0, 320, 3696, 2176), (1, 0, 4096, 256, 512), (1, 1, 4480, 256, 512), (1, 0, 1024, 128, 128), (1, 0, 512, 3200, 512), (1, 1, 512, 5760, 256),
]
# products in one piece with outer blocks, planned with 256 x 128 or 128 x 256 tiles that 128 x 128 ones take once blocked (dX, then dW, some ending inside a planned tile)
RETILED = [(1, 0, 5504, 1024, 256), (1, 1, 4224, 1408, 512), (1, 0, 256, 1024, 5504), (1, 1, 512, 1408, 4224),
           (1, 0, 640, 11264, 768)]
# long strips of the column-wise quantizers (four and eight slabs of 16 rows a wave), the last of them cut short
LONG = [(0, 0, 8256, 5120, 1088), (0, 0, 12352, 2048, 3456), (0, 0, 8256, 1024, 3584)]


def _tensors(N, D, C, outer, seed):
    import paper_2510_27527_amd as tj
    B = tj.binding
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    new = lambda r, c, s: (torch.randn((r, c), generator=g, device="cuda") * s).bfloat16()  # noqa: E731
    Xq = tj.quantize(new(N, D, 1.0), 0, B.ROUND_RTN, outer=outer)
    Wq = tj.quantize(new(C, D, 0.02), 0, B.ROUND_RTN, outer=outer)
    return new(N, C, 1e-3), Xq, Wq


def _row_major(dY, Xq, Wq, seed, layer, outer, rht):
    """Q3 .. Q6 by the quantizer's own call"""
    import paper_2510_27527_amd as tj
    B = tj.binding

    def q(src, axis, k):
        rid = (layer * 16 + (7 if k in (3, 4) else 8)) if rht else None
        return tj.quantize(src, axis, B.ROUND_SR, outer=outer, seed=seed, tensor_id=layer * 16 + k, rht_id=rid)
    return q(dY, 0, 3), q(Wq, 1, 4), q(dY, 1, 5), q(Xq, 1, 6)


def _without_padding(nbytes, operands):
    """bytes of a call's workspace without the scale bytes that only whole 256 k need; rows and reduction of each operand"""
    up = lambda v: (v + 255) // 256 * 256  # noqa: E731
    return nbytes - sum(up(r * ((k + 255) // 256) * 16) - up(r * k // 16) for r, k in operands)


def _least_workspace(op, N, D, C, outer):
    import paper_2510_27527_amd as tj
    B = tj.binding
    x, w = [(N, C), (D, C)], [(C, N), (D, N)]
    return _without_padding(B.workspace_bytes(op, N, D, C, outer), {B.OP_LINEAR_BWD_DX: x, B.OP_LINEAR_BWD_DW: w}.get(op, x + w))


@pytest.mark.gpu
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("outer,rht,N,D,C", CASES + REACH + RETILED + LONG)
def test_gradients_of_blocked_operands(outer, rht, N, D, C, f32):
    import paper_2510_27527_amd as tj
    B = tj.binding
    if f32 and (outer, rht, N, D, C) in LONG:
        pytest.skip("the quantizers are the same for both output types")
    dt = B.OUT_F32 if f32 else B.OUT_BF16
    dY, Xq, Wq = _tensors(N, D, C, outer, 7)
    dX, dW = tj.linear_bwd(dY, Xq, Wq, 11, 5, dt, rht=bool(rht))
    q3, q4, q5, q6 = _row_major(dY, Xq, Wq, 11, 5, outer, rht)
    assert torch.equal(dX, tj.gemm_nt(q3, q4, dt))
    assert torch.equal(dW, tj.gemm_nt(q5, q6, dt))
    assert torch.equal(dX, tj.linear_bwd_dx(dY, Wq, 11, 5, dt, rht=bool(rht)))
    assert torch.equal(dW, tj.linear_bwd_dw(dY, Xq, 11, 5, dt, rht=bool(rht)))
    # a workspace without room for the blocked scale bytes
    ws = {op: tj.alloc_workspace(_least_workspace(op, N, D, C, outer)) for op in (B.OP_LINEAR_BWD, B.OP_LINEAR_BWD_DX, B.OP_LINEAR_BWD_DW)}
    assert all(w.numel() <= max(16, B.workspace_bytes(op, N, D, C, outer)) for op, w in ws.items())
    aX, aW = tj.linear_bwd(dY, Xq, Wq, 11, 5, dt, rht=bool(rht), ws=ws[B.OP_LINEAR_BWD])
    assert torch.equal(dX, aX) and torch.equal(dW, aW)
    assert torch.equal(dX, tj.linear_bwd_dx(dY, Wq, 11, 5, dt, rht=bool(rht), ws=ws[B.OP_LINEAR_BWD_DX]))
    assert torch.equal(dW, tj.linear_bwd_dw(dY, Xq, 11, 5, dt, rht=bool(rht), ws=ws[B.OP_LINEAR_BWD_DW]))


# The split layer: outer mode, transform, N, D_lo, D_hp, C; whether dX_lo and dX_hp, and dW_lo, run on blocked operands; the tile of their launch together; whether
# the outlier channels' product would take another kernel or splits if launched alone
SPLIT = [
    (0, 0, 64, 64, 320, 64, False, False, None, False), (0, 0, 256, 64, 160, 64, False, True, None, False), (0, 0, 2944, 384, 416, 512, True, False, None, False),
    (0, 0, 1600, 6208, 96, 1280, True, True, None, True), (0, 0, 256, 4736, 64, 512, True, True, (128, 128), False), (0, 0, 256, 4352, 704, 256, True, True, (128, 128), True),
    (0, 0, 256, 7232, 64, 512, True, True, (128, 192), False), (0, 0, 384, 6912, 96, 640, True, True, (128, 256), False), (0, 0, 384, 8000, 576, 320, True, True, (128, 256), True),
    (0, 0, 448, 6336, 64, 320, True, True, (256, 128), False), (0, 0, 320, 5760, 192, 320, True, True, (256, 128), True), (0, 0, 448, 7488, 192, 640, True, True, (256, 256), True),
    (1, 0, 128, 128, 64, 128, False, False, None, False), (1, 0, 256, 128, 736, 128, False, True, None, False), (1, 1, 128, 128, 256, 2304, True, False, None, True),
    (1, 0, 256, 128, 448, 2048, True, True, None, True), (1, 0, 256, 1792, 640, 256, False, False, (64, 128), False), (1, 0, 512, 3072, 640, 512, True, True, (128, 128), False),
    (1, 1, 1280, 2304, 864, 1024, True, True, (128, 128), True), (1, 1, 512, 5760, 384, 256, True, True, (128, 192), False), (1, 0, 768, 3328, 832, 768, True, True, (128, 192), True),
    (1, 0, 512, 6016, 416, 512, True, True, (256, 128), False), (1, 1, 1024, 3072, 800, 768, True, True, (256, 128), True),
]


@pytest.mark.parametrize("outer,rht,N,D,H,C,x,w,tile,other", SPLIT)
def test_split_layers_run_on_the_stated_operands(outer, rht, N, D, H, C, x, w, tile, other):
    import paper_2510_27527_amd.binding as B
    lo, dw, hp = (B.backward_product_plan(B.OP_LINEAR_BWD, N, D, H, C, outer, k) for k in range(3))
    assert (lo.blocked, dw.blocked, hp.blocked) == (x, w, x)
    assert {lo.together, dw.together, hp.together} == {tile is not None} and (tile is None or lo.tile == tile)
    assert (B.gemm_splits_waves(N, H, C, outer) or B.gemm_plan(N, H, C, outer)[2] > 1) == other


@pytest.mark.gpu
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("outer,rht,N,D,H,C,x,w,tile,other", SPLIT)
def test_gradients_of_the_split_layer(outer, rht, N, D, H, C, x, w, tile, other, f32):
    """Byte for byte the gradients of a workspace that keeps the operands row-major, and the products of the quantizers' own row-major operands; where the
    launch together changes the outlier channels' kernel, and with it the order of summation, those within the products' tolerance."""
    import paper_2510_27527_amd as tj
    B = tj.binding
    dt = B.OUT_F32 if f32 else B.OUT_BF16
    dY, Xq, Wq = _tensors(N, D, C, outer, 9)
    g = torch.Generator(device="cuda")
    g.manual_seed(10)
    Xh, Wh = ((torch.randn((r, H), generator=g, device="cuda") * s).bfloat16() for r, s in ((N, 30.0), (C, 0.02)))
    got = tj.outctl_bwd(dY, Xq, Wq, Xh, Wh, 11, 5, dt, rht=bool(rht))
    size = B.lib().nvfp4_outctl_workspace_bytes(1, N, D, H, C, outer, dt)
    least = _without_padding(size, [(N, C), (D, C), (H, C), (C, N), (D, N)])
    assert (least < size) == (N % 256 != 0 or C % 256 != 0)
    for name, a, b in zip(("dX_lo", "dX_hp", "dW_lo", "dW_hp"), got, tj.outctl_bwd(dY, Xq, Wq, Xh, Wh, 11, 5, dt, rht=bool(rht), ws=tj.alloc_workspace(least))):
        assert torch.equal(a, b), name
    q3, q4, q5, q6 = _row_major(dY, Xq, Wq, 11, 5, outer, rht)
    q9 = tj.quantize(Wh, 1, B.ROUND_SR, outer=outer, seed=11, tensor_id=5 * 16 + 9, rht_id=5 * 16 + 7 if rht else None)
    assert torch.equal(got[0], tj.gemm_nt(q3, q4, dt)) and torch.equal(got[2], tj.gemm_nt(q5, q6, dt))
    if tile is None or not other:
        assert torch.equal(got[1], tj.gemm_nt(q3, q9, dt))
    else:
        ref = tj.gemm_nt(q3, q9, B.OUT_F32).double()
        near = 1e-3 if f32 else 2.0 ** -8
        # sums of C terms in another order, of operands whose products add up to some 1 / sqrt(C) of the sum of their sizes
        assert torch.all((got[1].double() - ref).abs() <= near * ref.abs() + 1e-6 * C ** 0.5 * ref.square().mean().sqrt())


def _plans(outer, N, D, C):
    """dX and dW of the call for both and of the two separate calls"""
    import paper_2510_27527_amd.binding as B
    plan = lambda op, product: B.backward_product_plan(op, N, D, 0, C, outer, product)  # noqa: E731
    return [(plan(B.OP_LINEAR_BWD, 0), C), (plan(B.OP_LINEAR_BWD, 1), N), (plan(B.OP_LINEAR_BWD_DX, 0), C), (plan(B.OP_LINEAR_BWD_DW, 1), N)]


def _blocked_launches(outer, N, D, C):
    """the instantiations of the product kernel that a layer's backward calls run on blocked operands"""
    out = set()
    for p, K in _plans(outer, N, D, C):
        if p.blocked:
            assert not p.split_waves
            out.add((outer, p.tile, "together" if p.together else "split" if p.split > 1 else "alone", N % 256 == C % 256 == 0 if p.together else K % 256 == 0))
    return out


def test_cases_reach_every_blocked_launch():
    """The planner's own answers for the launches of the table: among 6000 random layers there is no launch on blocked operands whose kernel the table
    does not run, every remainder of a reduction is there, and calls that block one product, both and none."""
    import paper_2510_27527_amd.binding as B
    table = CASES + REACH + RETILED + LONG
    have = set().union(*(_blocked_launches(o, N, D, C) for o, _, N, D, C in table))
    assert len(have) >= 41
    assert not {k for k in have if k[0] == 1 and k[1] in ((256, 128), (128, 256)) and k[2] == "alone"}    # 128 x 128 takes their place
    rng = random.Random(17)
    size = lambda lo, hi, step: step * max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step))  # noqa: E731
    for _ in range(6000):
        outer = rng.randint(0, 1)
        u = 128 if outer else 64
        N, D, C = size(u, 16384, u), size(128 if outer else 16, 8192, 128 if outer else 16), size(u, 8192, u)
        assert _blocked_launches(outer, N, D, C) <= have, (outer, N, D, C)
    for outer, remainders in ((0, {0, 64, 128, 192}), (1, {0})):
        assert {K % 256 for o, _, N, D, C in table if o == outer for p, K in _plans(o, N, D, C)[:2] if p.blocked} == remainders
        both = {tuple(p.blocked for p, _ in _plans(o, N, D, C)[:2]) for o, _, N, D, C in table if o == outer}
        assert {(True, True), (False, False), (True, False), (False, True)} <= both


@pytest.mark.parametrize("outer", [0, 1])
def test_products_with_a_launch_of_their_own_are_blocked_for_themselves(outer):
    """Only products that share a launch need one layout for all of them.  Without one, the call for both gradients blocks a product's operands where the
    separate call does (with per-tensor scales also dX's where that does not: it has no row-wise quantizer), and launches it alike; with outlier channels dX's
    two parts share an operand."""
    import paper_2510_27527_amd.binding as B
    rng = random.Random(29)
    size = lambda lo, hi, step: step * max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step))  # noqa: E731
    apart = 0
    for _ in range(1500):
        u = 128 if outer else 64
        N, D, C, H = size(u, 16384, u), size(u, 8192, u), size(u, 8192, u), size(32, 1024, 32)
        x, w, x0, w0 = (p for p, _ in _plans(outer, N, D, C))
        if not x.together:
            assert w == w0 and (x == x0 or not outer and x.blocked and not x0.blocked), (N, D, C)
            apart += x.blocked != w.blocked
        xl, wl, xh = (B.backward_product_plan(B.OP_LINEAR_BWD, N, D, H, C, outer, k) for k in range(3))
        if not xl.together:
            assert wl == w0 and xl.blocked == xh.blocked and x0.blocked >= xl.blocked, (N, D, H, C)
    assert apart >= 100


@pytest.mark.parametrize("op", ["dX", "dW", "both"])
def test_calls_that_lose_by_blocked_operands_keep_them_row_major(op):
    """calls that were measured to take longer with blocked operands, and on the other side of each line one that takes less (a product that can be blocked each time)"""
    import paper_2510_27527_amd.binding as B
    keep = {"dX": [(0, 65536, 256, 128), (0, 32768, 256, 320), (0, 1024, 64, 768), (1, 1792, 256, 256), (1, 512, 6656, 1280), (1, 7680, 2304, 256), (1, 256, 128, 1536)],
            "dW": [(0, 192, 4672, 4736), (1, 256, 2048, 256)], "both": [(0, 65536, 256, 64), (1, 256, 2944, 512)]}[op]
    take = {"dX": [(0, 16384, 512, 576), (1, 2048, 5632, 1536), (1, 256, 128, 2816), (1, 65536, 128, 256)], "dW": [(0, 320, 3008, 768), (1, 1024, 1152, 2048)],
            "both": [(0, 65536, 256, 256), (1, 1280, 2688, 1280)]}[op]
    which, product = {"dX": (B.OP_LINEAR_BWD_DX, 0), "dW": (B.OP_LINEAR_BWD_DW, 1), "both": (B.OP_LINEAR_BWD, 0)}[op]
    for layers, blocked in ((keep, False), (take, True)):
        for outer, N, D, C in layers:
            assert B.backward_product_plan(which, N, D, 0, C, outer, product).blocked == blocked, (outer, N, D, C)


@pytest.mark.parametrize("outer,rht,N,D,C", RETILED)
def test_retiled_cases_are_planned_otherwise(outer, rht, N, D, C):
    import paper_2510_27527_amd.binding as B
    seen = 0
    for (p, K), (M, Nn) in zip(_plans(outer, N, D, C), ((N, D), (C, D)) * 2):
        if p.blocked and not p.together and B.gemm_plan(M, Nn, K, outer) in ((256, 128, 1), (128, 256, 1)):
            assert p.tile == (128, 128) and p.split == 1
            seen += 1
    assert seen
