"""A ReLU layer keeps one order of summation.

Its gradient is a whole term where z > 0 and none where z <= 0: a z within
rounding of zero that changes sides with the order of its sum changes the
gradients by a term. So z is summed by the fp32 instructions, pair (k, k + 4)
after pair within each group of 8, one rounding per product."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2602_00125_amd import binding as b  # noqa: E402
DEV = "cuda:0"


def in_order(x, w):
    """sum_k x[k] w[k] in that order. The products of floats are exact in the
    64 bits of a long double; its sum, rounded again to 24 bits, is the fused
    multiply-add's but for one double rounding in 2^40."""
    K = len(x)
    s = np.float32(0)
    for g in range(0, K, 8):
        for j in range(4):
            for k in (g + j, g + 4 + j):
                if k < K:
                    s = np.float32(np.longdouble(x[k]) * np.longdouble(w[k]) + np.longdouble(s))
    return s


def layer(M, N, K, dtype=torch.float32, act="relu"):
    g = torch.Generator().manual_seed(M + K)
    x, w = torch.randn(M, K, generator=g).to(dtype), (torch.randn(N, K, generator=g) / K ** 0.5).to(dtype)
    bias = torch.randn(N, generator=g) / K ** 0.5
    y, z = (torch.full((M, N), float("nan"), device=DEV) for _ in range(2))
    b.linear_act_fwd(x.to(DEV), w.to(DEV), bias.to(DEV), act, y, z)
    y1 = torch.full_like(y, float("nan"))
    b.linear_act_fwd(x.to(DEV), w.to(DEV), bias.to(DEV), act, y1)
    assert torch.equal(y, y1)  # saving z does not change y
    return x, w, bias, y, z


# the classifier's hidden layer, ragged sizes without 16-byte rows, few rows,
# a contraction shorter than a stage
@pytest.mark.parametrize("M,N,K", [(512, 1024, 784), (777, 333, 509), (16, 4096, 256), (65, 64, 5)])
def test_saved_z_is_summed_in_order(M, N, K):
    x, w, bias, y, z = layer(M, N, K)
    z = z.cpu()
    assert torch.equal(y.cpu(), z.clamp(min=0))
    rng = np.random.default_rng(0)
    # random elements and those next to zero
    pos = [(int(rng.integers(M)), int(rng.integers(N))) for _ in range(24)]
    pos += [(int(i) // N, int(i) % N) for i in z.abs().flatten().argsort()[:24]]
    for m, n in pos:
        want = np.float32(in_order(x[m].numpy(), w[n].numpy()) + np.float32(bias[n]))
        assert np.float32(z[m, n]) == want, (m, n, float(z[m, n]), float(want))


# the ring tiles of large layers start their contraction at another stage on
# each XCD, so they are held to the forced tile instead; 128x128 and 256x256
# with 16-byte rows, 128x128 without; bf16 too
@pytest.mark.parametrize("M,N,K,cfg", [(2048, 1024, 256, 10), (4096, 4096, 64, 6), (2001, 1001, 100, 3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_saved_z_of_a_large_layer_takes_its_tile(M, N, K, cfg, dtype):
    z = layer(M, N, K, dtype)[4]
    try:
        b.debug_set("cfg", cfg)
        want = layer(M, N, K, dtype)[4]
    finally:
        b.debug_set("cfg", -1)
    assert torch.equal(z, want)
