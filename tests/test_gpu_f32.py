"""fp32-input products at the edges of their kernels: tiles and remainders,
16-byte and element-wise loads, split reductions, leading dimensions beyond
the matrix-core kernel's, special values.

Integer inputs whose sums stay below 2^24 are exact in fp32 whatever the
order of the sums, so whole outputs must equal the fp64 product.
"""
import pytest
import torch

from paper_2301_06813_amd import linear, sbp

from helpers import say

pytestmark = pytest.mark.gpu
F32 = sbp.SBP_F32


def _ints(rows, cols, pad, off, seed):
    """Integers in [-4, 4] as a view at column `off` of NaN-filled storage."""
    g = torch.Generator().manual_seed(seed)
    big = torch.full((rows + 1, off + cols + pad), float("nan"), device="cuda")
    v = big[:rows, off:off + cols]
    v.copy_(torch.randint(-4, 5, (rows, cols), generator=g).float())
    return v


def _kernel_names(fn):
    sbp.sbp_profile_begin(8)
    try:
        fn()
    finally:
        names = [n for n, _ in sbp.sbp_profile_end(8)]
    return names


@pytest.mark.parametrize("pad,off", [(0, 0), (8, 4), (0, 1), (3, 0)],
                         ids=["tight", "padded", "odd-offset", "odd-ld"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (64, 128, 64), (65, 97, 130), (4, 4100, 12),
                                   (257, 1000, 129), (640, 31, 2048), (1536, 260, 1664)])
def test_f32_exact_edges(shape, pad, off):
    M, K, N = shape
    X, W, dY = (_ints(a, b, pad, off, 40 + i) for i, (a, b) in
                enumerate(((M, K), (K, N), (M, N))))
    L = linear.layouts("BB", 1, 0)
    Xd, Wd, dYd = (t.cpu().double() for t in (X, W, dY))
    want = {"fwd": Xd @ Wd, "bwd_data": dYd @ Wd.t(), "bwd_weight": Xd.t() @ dYd}
    for op, w in want.items():
        for acc in (False, True):
            say("f32", shape, pad, off, op, acc)
            guard = torch.full((w.shape[0] + 2, w.shape[1] + 3), 5.0, device="cuda")
            out = guard[1:-1, 1:-2]
            linear.run_L(op, L, X, W, dY, out, accumulate=acc)
            got = out.cpu().double()
            assert torch.equal(got, w + 5.0 if acc else w)
            out.fill_(5.0)
            assert bool((guard == 5.0).all())


@pytest.mark.parametrize("acc", [False, True], ids=["store", "add"])
@pytest.mark.parametrize("pad,off", [(0, 0), (0, 1), (3, 0)], ids=["tight", "odd-offset", "odd-ld"])
@pytest.mark.parametrize("m,n,k,splits", [(2052, 1540, 196, 1), (2051, 1537, 167, 1),
                                          (1028, 1028, 1028, 3), (1025, 1027, 1030, 3)], ids=str)
@pytest.mark.parametrize("op", range(3), ids=["fwd", "bwd_data", "bwd_weight"])
def test_f32_128_tiles(op, m, n, k, splits, pad, off, acc):
    # the 128 x 128 instances, cut by every edge: 16-byte and 4-byte loads, whole and
    # split reductions, plain and accumulating
    M, K, N = ((m, k, n), (m, n, k), (k, m, n))[op]
    X, W, dY = (_ints(a, b, pad, off, 60 + i) for i, (a, b) in
                enumerate(((M, K), (K, N), (M, N))))
    Xd, Wd, dYd = (t.double() for t in (X, W, dY))
    want = (Xd @ Wd, dYd @ Wd.t(), Xd.t() @ dYd)[op].cpu()
    guard = torch.full((m + 2, n + 3), 5.0, device="cuda")
    out = guard[1:-1, 1:-2]
    say("f32 128", op, m, n, k, splits, pad, off, acc)
    L = linear.layouts("BB", 1, 0)
    names = _kernel_names(lambda: linear.run_L(("fwd", "bwd_data", "bwd_weight")[op], L, X, W, dY,
                                               out, accumulate=acc))
    assert torch.equal(out.cpu().double(), want + 5.0 if acc else want)
    out.fill_(5.0)
    assert bool((guard == 5.0).all())
    assert names[0].startswith("gemm_f32_mfma_kernel<128, "), names
    contig = {0: (k, n), 1: (k, k), 2: (m, n)}[op]
    v = 4 if pad == off == 0 and not any(c % 4 for c in contig) else 1
    assert names[0].endswith(", %d, %d>" % (v, 2 if acc and splits == 1 else 0)), names
    assert (len(names) == 2) == (splits > 1), names


@pytest.mark.parametrize("acc", [False, True], ids=["store", "add"])
@pytest.mark.parametrize("M,K,N", [(1020, 1024, 4092), (1019, 1021, 4093)], ids=str)
def test_f32_backward_pair_on_128_tiles(M, K, N, acc):
    X, W, dY = (_ints(a, b, 0, 0, 70 + i) for i, (a, b) in enumerate(((M, K), (K, N), (M, N))))
    L = linear.layouts("BB", 1, 0)
    gx, gw = (torch.full((a + 2, b + 3), 5.0, device="cuda") for a, b in ((M, K), (K, N)))
    dX, dW = gx[1:-1, 1:-2], gw[1:-1, 1:-2]
    say("f32 pair 128", M, K, N, acc)
    names = _kernel_names(lambda: linear.run_bwd_L(L, X, W, dY, dX, dW, accumulate_dw=acc))
    want = dY.double() @ W.double().t(), X.double().t() @ dY.double()
    assert torch.equal(dX.double(), want[0])
    assert torch.equal(dW.double(), want[1] + 5.0 if acc else want[1])
    dX.fill_(5.0)
    dW.fill_(5.0)
    assert bool((gx == 5.0).all()) and bool((gw == 5.0).all())
    assert names[0] == "gemm_f32_mfma_bwd_kernel<128, %d, %d>" % (4 if K % 4 == 0 else 1, acc), names


def test_f32_plans_reach_both_tiles_and_splits():
    plans = [sbp.sbp_plan(0, m, n, k, F32, F32) for m, n, k in
             ((1536, 1664, 260), (2048, 2048, 256), (4096, 4096, 512), (4, 12, 4100))]
    assert {p[0] for p in plans} == {64, 128}
    assert min(p[2] for p in plans) == 1 and max(p[2] for p in plans) > 1
    assert all(p[3] == sbp.KERNEL_F32 for p in plans)


@pytest.mark.parametrize("M,K,N,op,acc,kernel", [
    # stores bound these: the FMA kernel, unless they are added to the output
    (2100, 8, 2052, "fwd", False, "gemm_f32_kernel"), (2100, 12, 2052, "fwd", False, "64"),
    (1031, 12, 1025, "fwd", False, "gemm_f32_kernel"), (1031, 13, 1025, "fwd", False, "64"),
    (1031, 12, 1025, "fwd", True, "64"), (12, 123, 82, "bwd_weight", False, "gemm_f32_kernel"),
    (13, 123, 82, "bwd_weight", False, "64"), (12, 124, 84, "bwd_weight", False, "64"),
    (12, 123, 82, "bwd_weight", True, "64"), (12, 82, 123, "fwd", False, "64"),
    # a few steps of a 128 x 128 tile are bound by its stores
    (2048, 160, 2048, "fwd", False, "64"), (2048, 161, 2048, "fwd", False, "128")], ids=str)
def test_f32_short_reductions(M, K, N, op, acc, kernel):
    X, W, dY = (_ints(a, b, 0, 0, 90 + i) for i, (a, b) in enumerate(((M, K), (K, N), (M, N))))
    L = linear.layouts("BB", 1, 0)
    Xd, Wd, dYd = (t.cpu().double() for t in (X, W, dY))
    want = Xd @ Wd if op == "fwd" else Xd.t() @ dYd
    out = torch.full(want.shape, 5.0, device="cuda")
    names = _kernel_names(lambda: linear.run_L(op, L, X, W, dY, out, accumulate=acc))
    assert torch.equal(out.cpu().double(), want + 5.0 if acc else want)
    form = "gemm_f32_mfma_kernel<%s, " % kernel if kernel.isdigit() else kernel + "<"
    assert names[0].startswith(form), names
    if kernel.isdigit():   # the plain form holds no accumulating code
        assert names[0].endswith(", 2>" if acc else ", 0>"), names


def test_f32_leading_dimension_beyond_buffer_offsets():
    ld = (1 << 21) + 4
    X = torch.randint(-4, 5, (3, ld), device="cuda").float()[:, :70]
    W = torch.randint(-4, 5, (70, 40), device="cuda").float()
    out, _ = linear.call("fwd", "BB", 1, 0, X, W, None)
    assert torch.equal(out.cpu().double(), X.cpu().double() @ W.cpu().double())


def test_f32_special_values_stay_in_their_row():
    X = torch.ones(70, 66)
    X[3, 5], X[9, 65], X[69, 0] = float("inf"), float("nan"), -float("inf")
    X[20, :] = 1e-40   # subnormal inputs and products
    W = torch.rand(66, 70) + 1
    out = linear.call("fwd", "BB", 1, 0, X.cuda(), W.cuda(), None)[0].cpu()
    assert torch.isposinf(out[3]).all() and torch.isneginf(out[69]).all()
    assert torch.isnan(out[9]).all()
    rest = [i for i in range(70) if i not in (3, 9, 69)]
    want = (X.double() @ W.double())[rest]
    # 66 fp32 roundings, each at most 2^-24 of a partial sum of positive terms,
    # and at most half the smallest subnormal (2^-150) absolutely
    err = (out[rest].double() - want).abs()
    assert bool((err <= 66 * (2.0 ** -24 * want + 2.0 ** -149)).all())


@pytest.mark.parametrize("off", [0, 1], ids=["aligned", "odd-offset"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (64, 128, 64), (65, 97, 130), (4, 4100, 12),
                                   (1536, 260, 1664), (1024, 2048, 512)])
def test_f32_backward_pair(shape, off):
    # both products in one launch (where the plan groups them) and in two
    M, K, N = shape
    X, W, dY = (_ints(a, b, 0, off, 80 + i) for i, (a, b) in
                enumerate(((M, K), (K, N), (M, N))))
    L = linear.layouts("BB", 1, 0)
    want_dx = dY.cpu().double() @ W.cpu().double().t()
    want_dw = X.cpu().double().t() @ dY.cpu().double()
    for mode in (0, 1):
        for acc in (False, True):
            say("f32 pair", shape, off, mode, acc)
            gx, gw = (torch.full((a + 2, b + 3), 5.0, device="cuda") for a, b in ((M, K), (K, N)))
            dX, dW = gx[1:-1, 1:-2], gw[1:-1, 1:-2]
            try:
                sbp.sbp_set_bwd_override(mode, 1)
                names = _kernel_names(lambda: linear.run_bwd_L(L, X, W, dY, dX, dW,
                                                               accumulate_dw=acc))
            finally:
                sbp.sbp_set_plan_override(0, 0, 1)
            # the model groups all of these
            assert names[0].startswith("gemm_f32_mfma_bwd_kernel<") == (mode == 0), names
            assert torch.equal(dX.cpu().double(), want_dx)
            assert torch.equal(dW.cpu().double(), want_dw + 5.0 if acc else want_dw)
            dX.fill_(5.0)
            dW.fill_(5.0)
            assert bool((gx == 5.0).all()) and bool((gw == 5.0).all())
