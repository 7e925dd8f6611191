"""The generic bf16 kernel (operands at any element alignment) at the edges of
its tiles: chunks cut by the end of a row, the operand's last row, reduction
remainders, rows shorter than one 16-byte load, split reductions, unaligned
output rows.

The operands sit in NaN-filled storage, so an element read past a row that
reached a stored output would show. Integer inputs whose sums stay below 2^24
are exact in fp32 whatever the order of the sums.
"""
import pytest
import torch

from paper_2301_06813_amd import linear, sbp

from helpers import say

pytestmark = pytest.mark.gpu


def _ints(rows, cols, gap, off, seed):
    """Integers in [-3, 3], rows `gap` apart (odd row stride) at column off."""
    g = torch.Generator().manual_seed(seed)
    ld = off + cols + gap
    ld += 1 - ld % 2
    # the last row ends with the storage: nothing readable follows it
    flat = torch.full(((rows - 1) * ld + off + cols,), float("nan"), dtype=torch.bfloat16,
                      device="cuda")
    v = flat.as_strided((rows, cols), (ld, 1), off)
    v.copy_(torch.randint(-3, 4, (rows, cols), generator=g).to(torch.bfloat16))
    return v


@pytest.mark.parametrize("tile", [None, (256, 128), (128, 256), (128, 128), (128, 64), (64, 128),
                                  (64, 64)], ids=str)
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 7, 3), (64, 64, 128), (130, 63, 65),
                                   (127, 65, 129), (257, 193, 261), (72, 1000, 9)])
def test_generic_exact_edges(shape, tile):
    M, K, N = shape
    L = linear.layouts("BB", 1, 0)
    for gap, off in ((0, 0), (6, 3)):
        X, W, dY = (_ints(a, b, gap, off, 60 + i) for i, (a, b) in
                    enumerate(((M, K), (K, N), (M, N))))
        Xd, Wd, dYd = (t.cpu().double() for t in (X, W, dY))
        want = {"fwd": Xd @ Wd, "bwd_data": dYd @ Wd.t(), "bwd_weight": Xd.t() @ dYd}
        for op, w in want.items():
            for dtype, splits in ((torch.float32, 1), (torch.float32, 3), (torch.bfloat16, 1)):
                if dtype == torch.bfloat16 and op != "fwd":
                    continue   # partial sums are fp32
                say("generic", shape, tile, gap, off, op, dtype, splits)
                guard = torch.full((w.shape[0] + 2, w.shape[1] + 3), 7.0, dtype=dtype,
                                   device="cuda")
                out = guard[1:-1, 1:-2]
                if tile:
                    sbp.sbp_set_plan_override(*tile, splits, sbp.KERNEL_GENERIC)
                try:
                    linear.run_L(op, L, X, W, dY, out)
                finally:
                    sbp.sbp_set_plan_override(0, 0, 1)
                got = out.cpu().clone()
                assert torch.equal(got, w.to(dtype))
                out.fill_(7.0)
                assert bool((guard == 7.0).all())


@pytest.mark.parametrize("width", range(1, 8))
def test_generic_rows_narrower_than_a_load(width):
    # N = width: W and dY (and the output) have rows shorter than one 16-byte
    # load, tight or apart, over reductions that end in and around a whole step;
    # as K they make X narrow in the backward-weight product. Splits put the
    # rows near the operand's end into a reduction range of their own.
    L = linear.layouts("BB", 1, 0)
    g = torch.Generator().manual_seed(width)

    def ints(rows, cols, ld):
        flat = torch.full(((rows - 1) * ld + cols,), float("nan"), dtype=torch.bfloat16,
                          device="cuda")
        v = flat.as_strided((rows, cols), (ld, 1))
        v.copy_(torch.randint(-3, 4, (rows, cols), generator=g).to(torch.bfloat16))
        return v

    for red in (63, 64, 65, 70, 71, 72, 129, 199, 320):
        for ld in (width, width + 9):
            for splits in (1, 2):
                # forward: X 70 x red, W red x width; backward-weight: X red x
                # width (m-major), dY red x 75
                X, W = ints(70, red, red + 1 - red % 2), ints(red, width, ld)
                X2, dY2 = ints(red, width, ld), ints(red, 75, 75)
                for op, args, want in (("fwd", (X, W, None), (X, W)),
                                       ("bwd_weight", (X2, None, dY2), (X2.t(), dY2))):
                    say("narrow", width, red, ld, splits, op)
                    w = want[0].cpu().double() @ want[1].cpu().double()
                    guard = torch.full((w.shape[0] + 2, w.shape[1] + 3), 7.0, device="cuda")
                    out = guard[1:-1, 1:-2]
                    sbp.sbp_set_plan_override(64, 64, splits, sbp.KERNEL_GENERIC)
                    try:
                        linear.run_L(op, L, *args, out)
                    finally:
                        sbp.sbp_set_plan_override(0, 0, 1)
                    assert torch.equal(out.cpu().double(), w)
                    out.fill_(7.0)
                    assert bool((guard == 7.0).all())


def _graph_us(fn, calls=10, reps=9):
    """Median time of fn() in us, replayed from a graph."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            fn()
    t = []
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        graph.replay()
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(t)[reps // 2]


def test_narrow_rows_keep_the_loads_ahead():
    # an output 7 wide takes the plan and the steps of one 9 wide, and so its
    # time; with every step of the short rows loaded and computed in turn it took
    # 1.8 times as long
    ws = torch.empty(sbp.SBP_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")
    L = linear.layouts("BB", 1, 0)
    us = {}
    for n in (7, 9):
        X = torch.randn(8192, 4096, device="cuda").bfloat16()
        W = torch.randn(4096, n, device="cuda").bfloat16()
        out = torch.empty(8192, n, device="cuda")
        us[n] = _graph_us(lambda: linear.run_L("fwd", L, X, W, None, out, ws=ws))
    say("narrow rows", us)
    assert us[7] < 1.4 * us[9]
