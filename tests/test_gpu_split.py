"""fp32 products on the bf16 matrix cores split every value in three bf16 parts.

What the split does not serve (infinities, NaN, values and sums near the
largest float) must come out as in fp32 arithmetic, and what it serves must be
no further from the exact sums than fp32 accumulation is: tiny values too,
also beside ordinary ones that meet a zero.
"""
from __future__ import annotations

import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2602_00125_amd import binding as b  # noqa: E402
DEV = "cuda:0"
# 256x256, 128x128 (two depths), 256x128, 128x256 with 16-byte lanes; with
# vec1 those and 256x192, 256x96, 64x384 with 4-byte lanes
CFGS = [(c, 0) for c in (6, 8, 9, 10, 12)] + [(c, 1) for c in (6, 8, 9, 10, 13, 14, 15)]
KINDS = ["inf", "nan", "huge", "tiny_rows", "tiny_rows_big_other", "zero_rows", "mixed", "mixed_cols",
         "subnormal", "big_sums"]


def spoil(x, w, kind):
    """Rows of x (and of w) of the kind; the rest stays as drawn."""
    if kind == "inf":
        x[37, 5], x[201, 7], w[3, 11] = math.inf, -math.inf, math.inf
    elif kind == "nan":
        x[130, 1] = math.nan
    elif kind == "huge":  # h rounds to infinity; the products stay finite
        x[64, 3], x[65, 4] = 3.4028e38, -3.4027e38
        w *= 1e-6
    elif kind == "tiny_rows":
        x[10:20] *= 1e-36
    elif kind == "tiny_rows_big_other":
        x *= 1e-36
        w *= 1e30
    elif kind == "mixed":  # an ordinary value in every row meets a zero; the rest is tiny
        x *= 1e-37
        w *= 1e30
        x[:, 0], w[:, 0] = 1.0, 0.0
    elif kind == "mixed_cols":  # the other way round, other magnitudes in each row
        w *= 10.0 ** -torch.linspace(30, 38, len(w))[:, None]
        x *= 1e29
        w[:, 7], x[:, 7] = -3.0, 0.0
    elif kind == "subnormal":
        x *= 1e-40
        w *= 1e30
    elif kind == "big_sums":  # finite, beyond the scaled accumulators
        x *= 1e18
        w[4:60] *= 1e18
    elif kind == "zero_rows":
        x[5:9] = 0.0
        w[2] = 0.0
    return x, w


def check(got, want, S, K, what):
    """As fp32 sums of K products: |got - want| <= c S u, c = 2 sqrt(K) + 4
    for roundings of random sign (u = 2^-24), and one tiny float for a result
    in the subnormal range; not finite exactly where the exact result is not."""
    got = got.double().cpu()
    fin = torch.isfinite(want)
    assert torch.equal(torch.isnan(got), torch.isnan(want)), what
    assert torch.equal(got[~fin & ~torch.isnan(want)], want[~fin & ~torch.isnan(want)]), what
    err = (got - want).abs()[fin]
    bound = ((2 * math.sqrt(K) + 4) * 2.0 ** -24 * S + 2.0 ** -126)[fin]
    assert bool((err <= bound).all()), f"{what}: {float((err / bound).max())}"


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("cfg,vec1", CFGS)
def test_products_of_values_the_split_does_not_serve(cfg, vec1, kind):
    M, N, K = 300, 200, 136
    g = torch.Generator().manual_seed(cfg)
    x, w = spoil(torch.randn(M, K, generator=g), torch.randn(N, K, generator=g), kind)
    y, dw, db = (torch.full(s, math.nan, device=DEV) for s in ((M, N), (M, N), (M,)))
    xt, wt = x.t().contiguous().to(DEV), w.t().contiguous().to(DEV)
    X, W = x.double(), w.double()
    want, S = X @ W.t(), X.abs() @ W.t().abs()
    dbw, dbs = X.sum(1), X.abs().sum(1)
    try:
        b.debug_set("cfg", cfg)
        b.debug_set("vec1", vec1)
        b.linear_fwd(x.to(DEV), w.to(DEV), None, y)  # NT
        check(y, want, S, K, "y")
        y.fill_(math.nan)
        b.linear_bwd(None, wt, x.to(DEV), y, None, None)  # NN: x @ (K x N)
        check(y, want, S, K, "dx")
        for splits in (1, 3):  # TN with the column sums of its first operand, whole and in runs
            b.debug_set("splits", splits)
            ws = torch.empty(max(1, b.linear_bwd_workspace(wt, None, xt, None, dw, db)), dtype=torch.uint8, device=DEV)
            b.linear_bwd(wt, None, xt, None, dw, db, workspace=ws)
            check(dw, want, S, K, f"dw in {splits}")
            check(db, dbw, dbs, K, f"db in {splits}")
    finally:
        b.debug_set("cfg", -1)
        b.debug_set("vec1", 0)
        b.debug_set("splits", 0)


@pytest.mark.parametrize("kind", ["inf", "tiny_rows"])
def test_persistent_blocks_recompute_their_tiles(kind):
    """One block per CU walks several 256x256 tiles: the tiles of a block
    whose check fails are all written again."""
    M, N, K = 4352, 4096, 64
    g = torch.Generator().manual_seed(1)
    x, w = spoil(torch.randn(M, K, generator=g), torch.randn(N, K, generator=g), kind)
    bias = torch.randn(N, generator=g)
    y = torch.full((M, N), math.nan, device=DEV)
    b.linear_fwd(x.to(DEV), w.to(DEV), bias.to(DEV), y)
    X, W = x.double(), w.double()
    check(y, X @ W.t() + bias.double(), X.abs() @ W.t().abs() + bias.double().abs(), K, "y")


@pytest.mark.parametrize("kind", ["inf", "tiny_rows_big_other"])
@pytest.mark.parametrize("stride", [1, 2])
def test_convolution_of_values_the_split_does_not_serve(kind, stride):
    """The gathering products, stream-K and the sub-pixel phases included."""
    n, C, H, CO = 2, 32, 20, 64
    g = torch.Generator().manual_seed(3)
    x, w = torch.randn(n, C, H, H, generator=g), torch.randn(CO, C, 3, 3, generator=g) / 17
    ho = (H + 2 - 3) // stride + 1
    dy = torch.randn(n, CO, ho, ho, generator=g)
    if kind == "inf":
        x[1, 3, 4, 5], dy[0, 7, 2, 2] = math.inf, -math.inf
    else:
        x, dy, w = x * 1e-36, dy * 1e-36, w * 1e30
    cl = torch.channels_last
    xd, wd, dyd = (t.to(DEV).contiguous(memory_format=cl) for t in (x, w, dy))
    y, dx, dw, db = torch.empty_like(dyd), torch.empty_like(xd), torch.empty_like(wd), torch.empty(CO, device=DEV)
    X, W, D = (t.double().requires_grad_() for t in (x, w, dy))

    def grads(a, k, d):
        a, k = a.detach().requires_grad_(), k.detach().requires_grad_()
        out = torch.nn.functional.conv2d(a, k, stride=stride, padding=1)
        ga, gk = torch.autograd.grad(out, (a, k), d)
        return out.detach(), ga, gk

    try:
        for sk in (0, 1, 2):  # 1: as chosen, the phases in one grid of 128x128 tiles
            b.debug_set("stream_k", sk)
            b.debug_set("sk_blocks", 5 if sk == 2 else 0)
            b.debug_set("phase_grid", sk)
            b.debug_set("cfg", 6 if sk == 2 else -1)
            k1 = max(b.conv2d_fwd_workspace(xd, wd, None, y, stride, 1),
                     b.conv2d_bwd_workspace(xd, wd, dyd, dx, dw, db, stride, 1))
            ws = torch.empty(max(1, k1), dtype=torch.uint8, device=DEV)
            b.conv2d_fwd(xd, wd, None, y, stride, 1, workspace=ws)
            b.conv2d_bwd(xd, wd, dyd, dx, dw, db, stride, 1, workspace=ws)
            if kind == "inf":
                # a padded tap is absent here and a zero there: only which results are not finite
                f, a, c = grads(X, W, D)
                for got, want in ((y, f), (dx, a), (dw, c)):
                    assert torch.equal(torch.isfinite(got).cpu(), torch.isfinite(want))
            else:
                want = grads(X, W, D)
                scale = grads(X.abs(), W.abs(), D.abs())
                for got, v, S, K in zip((y, dx, dw), want, scale, (C * 9, CO * 9, n * ho * ho)):
                    check(got, v.detach(), S, K, "conv")
    finally:
        for k, v in (("stream_k", 1), ("sk_blocks", 0), ("phase_grid", 1), ("cfg", -1)):
            b.debug_set(k, v)


@pytest.mark.parametrize("K,runs", [(64, 1), (4096, 1), (100352, 28)])
def test_no_further_from_exact_than_fp32_sums(K, runs):
    """dW = dY^T X of normal values, unsplit or in runs, on the 256x256 tile:
    the fp32 instructions were 1.4e-7, 1.15e-6 and 1.08e-6 off here."""
    g = torch.Generator(DEV).manual_seed(K)
    x, dy = (torch.randn(K, 256, generator=g, device=DEV) for _ in range(2))
    dw = torch.empty(256, 256, device=DEV)
    try:
        b.debug_set("cfg", 6)
        b.debug_set("splits", runs)
        ws = torch.empty(max(1, b.linear_bwd_workspace(x, None, dy, None, dw, None)), dtype=torch.uint8, device=DEV)
        b.linear_bwd(x, None, dy, None, dw, None, workspace=ws)
    finally:
        b.debug_set("cfg", -1)
        b.debug_set("splits", 0)
    want = dy.double().t() @ x.double()
    rel = float((dw.double() - want).norm() / want.norm())
    assert rel <= {64: 1.4e-7, 4096: 1.15e-6, 100352: 1.08e-6}[K], rel


# one call's relative error against 64 bits, no larger than with fp32
# instructions (bf16: than in sixteen runs of 256 terms): runs of an NT, an NN
# and a TN product, and the shares of the small kernel's waves
@pytest.mark.parametrize("what,M,N,K,bar", [
    ("da", 509, 257, 383, 4.46e-7), ("db", 509, 257, 383, 4.71e-7), ("dx", 137, 3720, 1506, 2.86e-7),
    ("dx", 24, 3264, 2643, 2.68e-7), ("dx", 833, 2808, 64, 2.50e-7), ("dx bf16", 300, 4096, 300, 1.153e-7),
    ("dw bf16", 3320, 76, 752, 1.105e-7)])
def test_no_further_from_exact_than_before_the_split(what, M, N, K, bar):
    g = torch.Generator(DEV).manual_seed(1)
    if what in ("da", "db"):  # gradients of a broadcast batch: M x N (contracted in b) x K columns
        P, Q = 16, 8
        a, w = (2 * torch.rand(s, generator=g, device=DEV) - 1 for s in ((P, 1, M, N), (1, Q, N, K)))
        dc = torch.randn(P, Q, M, K, generator=g, device=DEV)
        x, y = (dc, w.transpose(-1, -2)) if what == "da" else (a.transpose(-1, -2), dc)
        out = torch.empty_like(a if what == "da" else w)
        ws = torch.empty(max(1, b.matmul_workspace(x, y, out, reduce_into=True)), dtype=torch.uint8, device=DEV)
        b.matmul(x, y, out, reduce_into=True, workspace=ws)
        want = torch.matmul(x.double(), y.double().contiguous()).sum(1 if what == "da" else 0, keepdim=True)
    else:
        dt = torch.bfloat16 if "bf16" in what else torch.float32
        x, w, dy = (torch.randn(s, generator=g, device=DEV).to(dt) for s in ((M, K), (N, K), (M, N)))
        dx, dw = (torch.empty(M, K, device=DEV), None) if "dx" in what else (None, torch.empty(N, K, device=DEV))
        ws = torch.empty(max(1, b.linear_bwd_workspace(x, w, dy, dx, dw)), dtype=torch.uint8, device=DEV)
        b.linear_bwd(x, w, dy, dx, dw, workspace=ws)
        out, want = (dx, dy.double() @ w.double()) if "dx" in what else (dw, dy.double().t() @ x.double())
    rel = float((out.double() - want).norm() / want.norm())
    assert rel <= bar, rel


@pytest.mark.parametrize("kind", ["inf", "nan", "big_sums"])
@pytest.mark.parametrize("cfg,vec1", [(6, 0), (10, 0), (10, 1), (8, 1), (16, 0), (17, 0), (18, 0)])
def test_refused_values_through_every_epilogue(cfg, vec1, kind):
    """The pass by the fp32 instructions ends in the same epilogues: a
    nonlinearity with z, adding to the outputs, both gradients and db in one
    launch, kept and summed batch elements, runs. (K with and without a tail.)"""
    g = torch.Generator().manual_seed(cfg)
    M, N = 300, 200
    try:
        b.debug_set("cfg", cfg)
        b.debug_set("vec1", vec1)
        for K in (128, 77):
            x, w = spoil(torch.randn(M, K, generator=g), torch.randn(N, K, generator=g), kind)
            X, W = x.double(), w.double()
            want, S = X @ W.t(), X.abs() @ W.t().abs()
            bias = torch.randn(N, generator=g)
            z, h = (torch.full((M, N), math.nan, device=DEV) for _ in range(2))
            b.linear_act_fwd(x.to(DEV), w.to(DEV), bias.to(DEV), "gelu", h, z)
            check(z, want + bias.double(), S + bias.double().abs(), K, "z")
            fin = torch.isfinite(z)
            near = torch.nn.functional.gelu(z.double())
            assert bool(((h.double() - near).abs() <= 1e-5 * z.double().abs() + 1e-6)[fin].all())
            # dY = x [M x K], W = w^T [K x N], X = the same rows again
            dy, wt = x.to(DEV), w.t().contiguous().to(DEV)
            xs = torch.randn(M, N, generator=g)
            prior = torch.randn(M, N, generator=g), torch.randn(K, N, generator=g), torch.randn(K, generator=g)
            wdw, Sdw = X.t() @ xs.double(), X.t().abs() @ xs.double().abs()
            for splits in (0, 3):
                b.debug_set("splits", splits)  # 0: a small cfg takes both gradients in one launch
                for acc in (False, True):
                    dx, dw, db = ((p if acc else torch.full_like(p, math.nan)).to(DEV) for p in prior)
                    ws = torch.empty(max(1, b.linear_bwd_workspace(xs.to(DEV), wt, dy, dx, dw, db)), dtype=torch.uint8,
                                     device=DEV)
                    b.linear_bwd(xs.to(DEV), wt, dy, dx, dw, db, accumulate=acc, workspace=ws)
                    for got, v, s, p, n in ((dx, want, S, prior[0], K), (dw, wdw, Sdw, prior[1], M),
                                            (db, X.sum(0), X.abs().sum(0), prior[2], M)):
                        p = p.double() * acc
                        check(got, v + p, s + p.abs(), n, f"{splits} {acc}")
                # a batch of two kept and three summed elements
                A = torch.stack([torch.stack([x, x * 0.5, -x]) for _ in range(2)])
                B = torch.stack([torch.stack([w, w, w * 2]) for _ in range(2)])
                for red in (False, True):
                    c = torch.full((2, 1 if red else 3, M, N), math.nan, device=DEV)
                    At, Bt = A.to(DEV), B.to(DEV).transpose(-1, -2)
                    ws = torch.empty(max(1, b.matmul_workspace(At, Bt, c, reduce_into=red)), dtype=torch.uint8, device=DEV)
                    b.matmul(At, Bt, c, reduce_into=red, workspace=ws)
                    wc, Sc = A.double() @ B.double().transpose(-1, -2), A.double().abs() @ B.double().abs().transpose(-1, -2)
                    if red:
                        wc, Sc = wc.sum(1, keepdim=True), Sc.sum(1, keepdim=True)
                    check(c, wc, Sc, 3 * K if red else K, f"batch {red} {splits}")
            b.debug_set("splits", 0)
    finally:
        for k, v in (("cfg", -1), ("vec1", 0), ("splits", 0)):
            b.debug_set(k, v)


# (the larger ones would be planned on 256x256 tiles)
@pytest.mark.parametrize("cfg,M,N", [(c, 300, 200) for c in (-1, 4, 10, 12, 16, 18)] +
                         [(c, 4352, 4096) for c in (-1, 4, 10, 12)])
def test_sums_of_one_or_two_products_are_rounded_as_such(cfg, M, N):
    """K = 1 is the rounded product itself, K = 2 the fused multiply-add of the second."""
    g = torch.Generator().manual_seed(M)
    for K in (1, 2):
        x, w = torch.randn(M, 4, generator=g), torch.randn(N, 4, generator=g)
        xd, wd = x.to(DEV)[:, :K], w.to(DEV)[:, :K]
        y = torch.full((M, N), math.nan, device=DEV)
        try:
            b.debug_set("cfg", cfg)
            b.linear_fwd(xd, wd, None, y)
        finally:
            b.debug_set("cfg", -1)
        want = (xd[:, :1].double() * wd[:, 0].double()).float()
        dw, db = torch.full((M, N), math.nan, device=DEV), torch.full((M,), math.nan, device=DEV)
        try:  # the same as a TN product with the column sums of its first operand
            b.debug_set("cfg", cfg)
            b.linear_bwd(wd.t().contiguous(), None, xd.t().contiguous(), None, dw, db)
        finally:
            b.debug_set("cfg", -1)
        assert torch.equal(dw, y)
        assert float((db.double() - xd.double().sum(1)).abs().max()) <= 2.0 ** -22
        if K == 2:  # (a sum of 48-bit products in 64 bits, rounded again: off by one place in 2^28)
            want = (xd[:, 1:2].double() * wd[:, 1].double() + want.double()).float()
            assert float((y != want).float().mean()) < 1e-6
        else:
            assert torch.equal(y, want)


@pytest.mark.parametrize("n", [1, 2])
def test_weight_gradient_of_a_convolution_over_one_or_two_pixels(n):
    g = torch.Generator().manual_seed(n)
    cl = torch.channels_last
    x, w, dy = (torch.randn(s, generator=g).to(DEV).contiguous(memory_format=cl)
                for s in ((n, 64, 3, 3), (96, 64, 3, 3), (n, 96, 1, 1)))
    dw, db = torch.full_like(w, math.nan), torch.full((96,), math.nan, device=DEV)
    ws = torch.empty(max(1, b.conv2d_bwd_workspace(x, w, dy, None, dw, db)), dtype=torch.uint8, device=DEV)
    b.conv2d_bwd(x, w, dy, None, dw, db, workspace=ws)
    X, D = x.double().cpu(), dy.double().cpu().view(n, 96)
    want = torch.einsum("no,nchw->ochw", D, X)
    check(dw, want, torch.einsum("no,nchw->ochw", D.abs(), X.abs()), n, "dw")
    check(db, D.sum(0), D.abs().sum(0), n, "db")


@pytest.mark.parametrize("shape", [((0, 5, 0), (0, 7)), ((3, 5, 0), (0, 7))])
def test_empty_contractions_are_zero(shape):
    """(no term: neither the split nor the fp32 instructions have a stage)"""
    a, k = torch.empty(shape[0], device=DEV), torch.empty(shape[1], device=DEV)
    c = torch.full((*shape[0][:2], 7), math.nan, device=DEV)
    b.matmul(a, k, c)
    assert bool((c == 0).all())
    r = torch.full((1, 5, 7), math.nan, device=DEV)  # summed over the batch axis, empty or not
    b.matmul(torch.empty(shape[0][0], 5, 4, device=DEV).zero_(), torch.ones(shape[0][0], 4, 7, device=DEV), r, reduce_into=True)
    assert bool((r == 0).all())
