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
