"""Products too small for the ring tiles: one tile a block, its waves sharing
the contraction, operands loaded in place (any alignment)."""
from __future__ import annotations

import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2602_00125_amd import binding as b  # noqa: E402
from test_gpu_split import KINDS, check, spoil  # noqa: E402
DEV = "cuda:0"
TILES = {16: 64, 17: 32, 18: 16}
# every tile edge +-1 and short, whole, one-past and long contractions
SIZES = [(1, 1, 1), (1, 2, 33), (2, 1, 65), (3, 2, 31), (15, 17, 32), (16, 16, 64), (17, 63, 31), (64, 64, 96),
         (65, 33, 257), (130, 66, 40), (20, 300, 1000), (257, 31, 545)]


def close(got, want, S, K, what, u=2.0 ** -24):
    """|got - want| <= (2 sqrt(K) + 4) u S: K products, roundings of random sign."""
    got, err = got.double().cpu(), (got.double().cpu() - want).abs()
    bound = (2 * math.sqrt(K) + 4) * u * S + 2.0 ** -126
    assert bool(torch.isfinite(got).all()) and bool((err <= bound).all()), f"{what}: {float((err / bound).max())}"


@pytest.mark.parametrize("M,N,K", SIZES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cfg", [16, 17, 18, -1])
def test_layer(cfg, dtype, M, N, K):
    """Y (with bias, and with a nonlinearity), dX, dW and db, one by one and
    both gradients in one launch, overwriting and accumulating; operands at
    an odd offset and pitch."""
    g = torch.Generator().manual_seed(M * 7 + N)

    def view(r, c, odd):
        t = torch.randn(r, c + odd, generator=g).to(dtype)
        d = torch.empty(r * (c + odd) + 1, dtype=dtype, device=DEV)[odd:odd + r * (c + odd)].view(r, c + odd)
        d.copy_(t)
        return t[:, :c], d[:, :c]

    for odd in (0, 1):
        (x, xd), (w, wd), (dy, dyd) = view(M, K, odd), view(N, K, odd), view(M, N, odd)
        bias = torch.randn(N, generator=g)
        X, W, D = x.double(), w.double(), dy.double()
        z, h = (torch.full((M, N), math.nan, device=DEV) for _ in range(2))
        y = torch.full((M, N), math.nan, device=DEV)
        want = {"dx": (D @ W, D.abs() @ W.abs(), N), "dw": (D.t() @ X, D.t().abs() @ X.abs(), M),
                "db": (D.sum(0), D.abs().sum(0), M)}
        try:
            b.debug_set("cfg", cfg)
            b.linear_fwd(xd, wd, bias.to(DEV), y)
            b.linear_act_fwd(xd, wd, bias.to(DEV), "relu", h, z)
            Z, S = X @ W.t() + bias.double(), X.abs() @ W.t().abs() + bias.double().abs()
            close(y, Z, S, K, "y")
            close(z, Z, S, K, "z")
            assert torch.equal(h, z.clamp(min=0))
            for names in (("dx", "dw", "db"), ("dx",), ("dw", "db"), ("dx", "dw")):
                for acc in (False, True):
                    prior = {n: torch.randn(want[n][0].shape, generator=g) for n in names}
                    out = {n: (prior[n].to(DEV) if acc else torch.full(want[n][0].shape, math.nan, device=DEV)) for n in names}
                    b.linear_bwd(xd, wd, dyd, *(out.get(n) for n in ("dx", "dw", "db")), accumulate=acc)
                    for n in names:
                        v, s, k = want[n]
                        if acc:
                            v, s = v + prior[n].double(), s + prior[n].double().abs()
                        close(out[n], v, s, k, f"{n} of {names} acc={acc} odd={odd}")
        finally:
            b.debug_set("cfg", -1)


@pytest.mark.parametrize("cfg", [16, 17, 18])
@pytest.mark.parametrize("K", [33, 64])
def test_batched_and_summed(cfg, K):
    """Broadcast batches and the sums over them, in every operand layout
    (whole K-steps and a tail in each summed element), and stride-0 views."""
    g = torch.Generator().manual_seed(cfg)
    A, B = torch.randn(3, 1, 37, K, generator=g), torch.randn(1, 4, K, 41, generator=g)
    want, S = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    one = torch.randn(1, K, generator=g)
    try:
        b.debug_set("cfg", cfg)
        for ta in (False, True):
            for tb in (False, True):
                a = (A.mT.contiguous().to(DEV).mT if ta else A.to(DEV))
                w = (B.mT.contiguous().to(DEV).mT if tb else B.to(DEV))
                c = torch.full((3, 4, 37, 41), math.nan, device=DEV)
                b.matmul(a, w, c)
                close(c, want, S, K, f"c {ta} {tb}")
                c = torch.full((4, 37, 41), math.nan, device=DEV)
                b.matmul(a, w, c, reduce_into=True)
                close(c, want.sum(0), S.sum(0), 3 * K, f"sum {ta} {tb}")
        # every row of the first operand the same memory
        c = torch.full((4, 37, 41), math.nan, device=DEV)
        b.matmul(one.to(DEV).expand(37, K), B[0].to(DEV), c)
        close(c, one.double().expand(37, K) @ B[0].double(), one.double().abs() @ B[0].double().abs(), K, "expanded")
    finally:
        b.debug_set("cfg", -1)


@pytest.mark.parametrize("cfg", [16, 17, 18])
@pytest.mark.parametrize("kind", KINDS)
def test_values_the_split_does_not_serve(cfg, kind):
    g = torch.Generator().manual_seed(cfg)
    M, N, K = 210, 70, 136
    x, w = spoil(torch.randn(M, K, generator=g), torch.randn(N, K, generator=g), kind)
    y, db = torch.full((M, N), math.nan, device=DEV), torch.full((M,), math.nan, device=DEV)
    xt, wt = x.t().contiguous().to(DEV), w.t().contiguous().to(DEV)
    X, W = x.double(), w.double()
    want, S = X @ W.t(), X.abs() @ W.t().abs()
    try:
        b.debug_set("cfg", cfg)
        b.linear_fwd(x.to(DEV), w.to(DEV), None, y)
        check(y, want, S, K, "y")
        b.linear_bwd(None, wt, x.to(DEV), y.fill_(math.nan), None, None)
        check(y, want, S, K, "dx")
        b.linear_bwd(wt, None, xt, None, y.fill_(math.nan), db)
        check(y, want, S, K, "dw")
        check(db, X.sum(1), X.abs().sum(1), K, "db")
    finally:
        b.debug_set("cfg", -1)


def best_time(f):
    f()
    best = math.inf
    for _ in range(5):
        a, e = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(4):
            f()
        e.record()
        e.synchronize()
        best = min(best, a.elapsed_time(e))
    return best


@pytest.mark.parametrize("N", [1, 2, 3, 5])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_layers_of_a_few_outputs(N, dtype):
    """dW of a head of N outputs: rows of dY shorter than the tile's vectors,
    up to the matrix's last element (what follows is NaN) and no further, at
    remainders around a K-step; and its contraction is shared by the waves."""
    g = torch.Generator().manual_seed(N)
    K = 70
    try:
        for cfg in (16, 17, 18):
            b.debug_set("cfg", cfg)
            for M in (1, 2, 31, 32, 33, 34, 35, 64, 67, 97, 330):
                x, dy, w = (torch.randn(s, generator=g).to(dtype) for s in ((M, K), (M, N), (N, K)))
                buf = torch.full((M * N + 8,), math.nan, dtype=dtype, device=DEV)
                d = buf[:M * N].view(M, N)
                d.copy_(dy)
                X, D, W = x.double(), dy.double(), w.double()
                dx, dw, db = (torch.full(s, math.nan, device=DEV) for s in ((M, K), (N, K), (N,)))
                b.linear_bwd(x.to(DEV), w.to(DEV), d, dx, dw, db)
                close(dw, D.t() @ X, D.t().abs() @ X.abs(), M, f"dw {cfg} {M}")
                close(dx, D @ W, D.abs() @ W.abs(), N, f"dx {cfg} {M}")
                close(db, D.sum(0), D.abs().sum(0), M, f"db {cfg} {M}")
    finally:
        b.debug_set("cfg", -1)
    M, K = 8192, 1024

    def step(n):
        x, dy, w = (torch.randn(s, device=DEV).to(dtype) for s in ((M, K), (M, n), (n, K)))
        o = torch.empty(M, K, device=DEV), torch.empty(n, K, device=DEV), torch.empty(n, device=DEV)
        ws = torch.empty(max(1, b.linear_bwd_workspace(x, w, dy, *o)), dtype=torch.uint8, device=DEV)
        return best_time(lambda: b.linear_bwd(x, w, dy, *o, workspace=ws))

    # one wave walking 256 K-steps alone took 7 times as long as 64 outputs
    assert step(N) < 3 * step(64)


def test_runs_of_a_long_contraction():
    """A 16x16 weight gradient over 20000 rows: split over the grid when a
    workspace is given, whole without one; db in the same launch."""
    g = torch.Generator().manual_seed(2)
    x, dy = torch.randn(20000, 16, generator=g), torch.randn(20000, 16, generator=g)
    X, D = x.double(), dy.double()
    dw, db = torch.empty(16, 16, device=DEV), torch.empty(16, device=DEV)
    for ws in (None, torch.empty(1 << 22, dtype=torch.uint8, device=DEV)):
        b.linear_bwd(x.to(DEV), None, dy.to(DEV), None, dw.fill_(math.nan), db.fill_(math.nan), workspace=ws)
        close(dw, D.t() @ X, D.t().abs() @ X.abs(), 20000, "dw")
        close(db, D.sum(0), D.abs().sum(0), 20000, "db")


def test_convolution_weight_gradient_within_a_smaller_workspace():
    """49 runs where the workspace holds them; fewer, down to 16, where it does
    not (whole, it takes 18 times as long)."""
    N, C, H, W, CO = 16, 64, 56, 56, 128
    x, w, dy = (torch.randn(s, device=DEV).contiguous(memory_format=torch.channels_last)
                for s in ((N, C, H, W), (CO, C, 3, 3), (N, CO, 28, 28)))
    dw, db = torch.empty_like(w), torch.empty(CO, device=DEV)
    full = b.conv2d_bwd_workspace(x, w, dy, None, dw, db, 2, 1)
    X, K = x.double().cpu(), w.double().cpu().requires_grad_()
    out = torch.nn.functional.conv2d(X, K, stride=2, padding=1)
    want, = torch.autograd.grad(out, K, dy.double().cpu())
    S, = torch.autograd.grad(torch.nn.functional.conv2d(X.abs(), K, stride=2, padding=1), K, dy.double().cpu().abs())
    t = []
    for n in (full, full // 3):
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
        dw.fill_(math.nan), db.fill_(math.nan)
        t.append(best_time(lambda: b.conv2d_bwd(x, w, dy, None, dw, db, 2, 1, workspace=ws)))
        close(dw, want, S, N * 28 * 28, f"dw in {n} bytes")
        close(db, dy.double().cpu().sum((0, 2, 3)), dy.double().cpu().abs().sum((0, 2, 3)), N * 28 * 28, f"db in {n} bytes")
    assert t[1] < 4 * t[0], t


# outputs and sums around every group size (4, 16, 64 and 256 lanes), with
# and without 16-byte rows, one and several summed axes, views
REDUCTIONS = [((3, 5, 7), k) for k in ("a", "b", "c", "ab", "ac", "bc", "")] + \
             [((4, 3, 8), k) for k in ("a", "b", "c", "ab", "ac", "bc", "")] + \
             [((2, 130, 36), k) for k in ("a", "b", "c", "ab", "ac", "bc")] + \
             [((33, 2, 1028), k) for k in ("a", "b", "ab", "ac")] + [((1, 1, 20000), ""), ((700, 3, 40), "b"),
              ((5, 1, 4101), "a"), ((4096, 2, 4), "c"), ((2, 600, 260), "ac")]


@pytest.mark.parametrize("shape,keep", REDUCTIONS)
@pytest.mark.parametrize("view", ["whole", "pitch", "permuted", "expanded"])
def test_reduction(shape, keep, view):
    g = torch.Generator().manual_seed(sum(shape))
    t = torch.randn(shape, generator=g)
    x = t.to(DEV)
    if view == "pitch":
        x = torch.nn.functional.pad(x, (1, 2))[..., 1:-2]
    elif view == "permuted":
        x = x.permute(2, 0, 1).contiguous().permute(1, 2, 0)
    elif view == "expanded":
        t = t[:, :1].expand(shape)
        x = x[:, :1].expand(shape)
    axes = [i for i, a in enumerate("abc") if a not in keep]
    want = t.double().sum(axes, keepdim=True) if axes else t.double()
    S = t.double().abs().sum(axes, keepdim=True) if axes else t.double().abs()
    n = t.numel() // want.numel()
    for parts, acc in ((0, False), (0, True), (3, False)):
        b.debug_set("parts", parts)
        try:
            prior = torch.randn(want.shape, generator=g)
            out = prior.to(DEV) if acc else torch.full(want.shape, math.nan, device=DEV)
            k = b.reduce_broadcast_grad_workspace(x, out)
            for ws in (None, torch.empty(k, dtype=torch.uint8, device=DEV) if k else None):
                got = out.clone()
                b.reduce_broadcast_grad(x, got, accumulate=acc, workspace=ws)
                p = prior.double() if acc else torch.zeros_like(want)
                close(got, want + p, S + p.abs(), n, f"{parts} {acc} {ws is None}")
        finally:
            b.debug_set("parts", 0)


@pytest.mark.parametrize("n", [(1 << 24) - 1, (1 << 24) + 3])
def test_reduction_to_many_outputs_of_long_sums(n):
    """A block an output would be a launch of 2^32 threads."""
    row = torch.randn(4096, generator=torch.Generator().manual_seed(0))
    out = torch.full((n, 1), math.nan, device=DEV)
    b.reduce_broadcast_grad(row.to(DEV).expand(n, 4096), out)
    assert bool((out == out[0]).all())
    close(out[0], row.double().sum(), row.double().abs().sum(), 4096, "sum")


from test_gpu_conv import PHASE_CASES, check as conv_check, make as conv_make, run as conv_run  # noqa: E402


@pytest.mark.parametrize("case", PHASE_CASES, ids=[f"p{i}" for i in range(len(PHASE_CASES))])
def test_strided_input_gradient_in_one_grid_of_small_tiles(case):
    """Every sub-pixel phase in one grid of 128x128 tiles (the default for
    gradients that do not fill 256x256 ones), against the oracle."""
    x, w, bias, dy = conv_make(case, seed=73)
    conv_check(case, x, w, bias, dy, *conv_run(case, x, w, bias, dy))
    N, C, H, W, CO, KH, KW = case[:7]
    prior = (torch.randn(N, C, H, W, device=DEV), None, None)
    got = conv_run(case, x, w, bias, dy, outputs=("dx",), accumulate=True, prior=prior)
    conv_check(case, x, w, bias, dy, got[0], got[1], None, None, prior=prior)
