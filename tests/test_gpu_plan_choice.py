"""The plan that the time model chooses is near the fastest of the plans it chooses
among, for products whose choice was once wrong: accumulating outputs, outputs of a
few tiles, rows that are not whole 64-byte blocks, operands in the shifted form."""
import pytest
import torch

from paper_2301_06813_amd import linear, sbp

from helpers import say
from test_gpu_attn_group import INSTANCES
from test_gpu_generic import _graph_us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,sig,shape,acc", [
    ("bwd_weight", "DP", (896, 4160, 192), True), ("bwd_weight", "DP", (256, 2048, 576), True),
    ("bwd_weight", "DP", (64, 3712, 512), True), ("bwd_weight", "DP", (2048, 6016, 512), True),
    ("bwd_weight", "DP", (384, 192, 384), False), ("bwd_weight", "DP", (560, 1456, 424), False),
    ("fwd", "DP", (2592, 64, 4120), False), ("bwd_data", "COL", (6080, 192, 64), False),
    ("bwd_weight", "DP", (248, 2803, 1171), False), ("fwd", "DP", (785, 523, 2037), False),
    ("bwd_data", "COL", (1643, 1951, 238), False)], ids=str)
def test_chosen_plan_is_near_the_fastest(op, sig, shape, acc):
    M, K, N = shape
    # rows that start on 16-byte blocks
    X, W, dY = (torch.randn(a, -(-b // 8) * 8, device="cuda").bfloat16()[:, :b]
                for a, b in ((M, K), (K, N), (M, N)))
    L = linear.layouts(sig, 1, 0)
    out = linear.alloc_out_L(op, L, M, K, N, torch.bfloat16, "cuda")
    out = (out.float() if acc else out).zero_()
    ws = torch.empty(sbp.SBP_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")

    def us():
        return _graph_us(lambda: linear.run_L(op, L, X, W, dY, out, accumulate=acc, ws=ws))

    chosen = us()
    forced = {}
    try:
        for bm, bn, code in INSTANCES:
            for splits in (1, 2, 4):
                sbp.sbp_set_plan_override(bm, bn, splits, code)
                forced[bm, bn, code, splits] = us()
    finally:
        sbp.sbp_set_plan_override(0, 0, 1)
    best = min(forced, key=forced.get)
    say(op, shape, "chosen %.2f us, fastest %.2f us" % (chosen, forced[best]), best)
    # 15 % at the 99th percentile of the fit, and a tenth for noise; the choices that
    # this is about were 1.3 to 1.8 times the fastest
    assert chosen <= 1.25 * forced[best]
