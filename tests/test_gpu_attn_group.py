"""The attention backward calls as one grouped launch, on every instance the
planner may choose, at tile edges; the cases that stay two launches (outputs of
two types, operands the pipelined kernel cannot read, two launches asked for)
give the same results.

Integer inputs whose sums stay below 2^24 are exact in fp32; bf16 outputs are
compared with the product rounded to nearest even.
"""
import pytest
import torch

from paper_2301_06813_amd import sbp

from helpers import say

pytestmark = pytest.mark.gpu
INSTANCES = [(64, 64, 1), (64, 64, 4), (64, 64, 12), (64, 128, 4), (64, 128, 12), (128, 64, 4),
             (128, 64, 12), (128, 128, 4), (128, 128, 12), (256, 192, 1), (256, 256, 1)]


def _ints(shape, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-3, 4, shape, generator=g).to(torch.bfloat16).cuda()


def _out(b, h, n, d, dtype):
    """[b][h][n][d] stored [b][n][h][d], in a guarded buffer."""
    buf = torch.full((b + 1, n, h, d), 9.0, dtype=dtype, device="cuda")
    return buf, buf[:b].permute(0, 2, 1, 3)


def _check(b, h, sq, sk, d, dts, accumulate=False):
    Q, K, V, dO = (_ints((b, n, h, d), i).permute(0, 2, 1, 3)
                   for i, n in enumerate((sq, sk, sk, sq)))
    P, dS = _ints((b, h, sq, sk), 5), _ints((b, h, sq, sk), 6)
    D = {k: t.cpu().double() for k, t in dict(Q=Q, K=K, V=V, dO=dO, P=P, dS=dS).items()}
    want = {"dQ": D["dS"] @ D["K"], "dK": D["dS"].transpose(2, 3) @ D["Q"],
            "dP": D["dO"] @ D["V"].transpose(2, 3), "dV": D["P"].transpose(2, 3) @ D["dO"]}
    scope = sbp.SBP_ACCUMULATE if accumulate else sbp.SBP_LOCAL
    v = {k: sbp.view4(t) for k, t in dict(Q=Q, K=K, V=V, dO=dO, P=P, dS=dS).items()}
    bufs = {"dQ": _out(b, h, sq, d, dts[0]), "dK": _out(b, h, sk, d, dts[1]),
            "dV": _out(b, h, sk, d, dts[1])}
    dp = torch.full((b + 1, h, sq, sk), 9.0, dtype=dts[0], device="cuda")
    bufs["dP"] = (dp, dp[:b])
    o = {k: sbp.view4(t, scope) for k, (_, t) in bufs.items()}
    sbp.sbp_profile_begin(8)
    try:
        sbp.sbp_attn_scores_bwd(v["dS"], v["Q"], v["K"], o["dQ"], o["dK"], 1, 0)
        sbp.sbp_attn_context_bwd(v["dO"], v["P"], v["V"], o["dP"], o["dV"], 1, 0)
    finally:
        names = [n for n, _ in sbp.sbp_profile_end(8)]
    for k, (buf, t) in bufs.items():
        w = want[k] + (9.0 if accumulate else 0.0)
        assert torch.equal(t.cpu(), w.to(t.dtype)), k
        assert bool((buf[b:] == 9.0).all()), k
    return names


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("inst", INSTANCES, ids=lambda i: "%dx%d-k%d" % i)
def test_grouped_every_instance(inst, dtype):
    for dims in ((2, 3, 136, 72, 40), (1, 2, 64, 264, 128), (1, 1, 8, 8, 8)):
        say("attn grouped", inst, dims, dtype)
        try:
            sbp.sbp_set_plan_override(inst[0], inst[1], 1, inst[2])
            sbp.sbp_set_bwd_override(2, 1)
            for acc in (False, True) if dtype == torch.float32 else (False,):
                # one launch a call: of this tile, in the accumulating form or the plain one
                names = _check(*dims, (dtype, dtype), accumulate=acc)
                assert len(names) == 2, names
                for n in names:
                    assert n.startswith("gemm_bf16_dma_bwd_kernel<%d, %d, " % inst[:2]), names
                    assert n.endswith(", 1>") == acc, names
        finally:
            sbp.sbp_set_plan_override(0, 0, 1)


@pytest.mark.parametrize("dims", [(2, 3, 136, 72, 40), (1, 1, 200, 200, 64), (3, 2, 67, 33, 20),
                                  (2, 2, 64, 128, 96)], ids=str)
def test_default_plans_types_and_accumulation(dims):
    bf, f32 = torch.bfloat16, torch.float32
    for dts in ((bf, bf), (f32, f32), (bf, f32), (f32, bf)):
        say("attn default", dims, dts)
        _check(*dims, dts)
    _check(*dims, (f32, f32), accumulate=True)
    try:
        sbp.sbp_set_bwd_override(1, 1)   # two launches
        assert len(_check(*dims, (bf, bf))) == 4
    finally:
        sbp.sbp_set_plan_override(0, 0, 1)
