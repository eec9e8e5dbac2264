"""The work that is timed: calls of the public entry points over the sizes they are used at.

``listed()`` gives the cases, ``draw(rng)`` one more of the same ranges,
``prepare(case, seed)`` what a program holds before the call (inputs, output
buffers and workspaces on the GPU), ``run(state)`` one pass,
``exact(case, seed)`` the pass in 64 bits by plain torch, ``work(case)`` the
bytes and operations a pass cannot do without and ``tolerance(case)`` how far
another correct fp32 implementation may be from it.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2602_00125_amd import binding as mt

DEV = "cuda:0"
LR, BETA1, BETA2, EPS, STEP = 1e-3, 0.9, 0.999, 1e-8, 100  # an Adam run some way in


def listed():
    return [
        # a training step (forward, dX, dW, db) of one dense layer. The
        # smallest: bound by latency and launches
        dict(name="dense_64x32x128_f32", kind="dense", M=64, N=32, K=128, dtype="f32"),
        # odd sizes throughout: no row is 16-byte aligned
        dict(name="dense_777x1001x509_f32", kind="dense", M=777, N=1001, K=509, dtype="f32"),
        # an ordinary hidden layer
        dict(name="dense_4096x1024x1024_f32", kind="dense", M=4096, N=1024, K=1024, dtype="f32"),
        # the large layer the benchmark quotes
        dict(name="dense_8192x8192x8192_f32", kind="dense", M=8192, N=8192, K=8192, dtype="f32"),
        # bf16 operands: an ordinary layer and the largest
        dict(name="dense_2048x1536x1000_bf16", kind="dense", M=2048, N=1536, K=1000, dtype="bf16"),
        dict(name="dense_16384x8192x8192_bf16", kind="dense", M=16384, N=8192, K=8192, dtype="bf16"),
        # evaluation of a few rows: a dense layer and its nonlinearity, forward only
        dict(name="eval_16x4096x4096_f32_gelu", kind="eval", M=16, N=4096, K=4096, dtype="f32", act="gelu"),
        # broadcasting batched matmul with odd sizes, and both operands' gradients
        # summed over the axes they were broadcast along
        dict(name="bmm_16x8_509x257x383_f32", kind="bmm", P=16, Q=8, M=509, K=257, N=383),
        # a training step of a convolution mid-way through an image classifier,
        dict(name="conv_32x256x56x56_256x3x3_s1", kind="conv", N=32, C=256, H=56, W=56, CO=256, k=3, s=1, p=1,
             layout="cl"),
        # and a smaller one that halves the image
        dict(name="conv_16x64x56x56_128x3x3_s2", kind="conv", N=16, C=64, H=56, W=56, CO=128, k=3, s=2, p=1,
             layout="cl"),
        # a whole training step of a two-layer classifier on flattened 28 x 28
        # images: both layers, mean squared error, backward, Adam
        dict(name="mlp_512x784x1024x10_f32_relu", kind="mlp", M=512, D0=784, D1=1024, D2=10, act="relu"),
        # the gradient of a per-channel bias of a [batch, channel, position] tensor
        dict(name="unbroadcast_32x128x4096_channel", kind="unbroadcast", A=32, B=128, C=4096, keep="B"),
    ]


def _size(rng, lo, hi):
    """A size from lo to hi, spread over its logarithm; multiples of 64 or 8 about as often as any."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    g = rng.choice([64, 64, 8, 1])
    return int(min(hi, max(lo, round(v / g) * g)))


def draw(rng):
    kind = rng.choice(["dense"] * 6 + ["eval", "eval", "bmm", "bmm", "conv", "conv", "mlp", "unbroadcast"])
    if kind == "dense":
        return dict(kind=kind, M=_size(rng, 32, 8192), N=_size(rng, 16, 8192), K=_size(rng, 16, 8192),
                    dtype=rng.choice(["f32", "f32", "f32", "bf16"]))
    if kind == "eval":
        return dict(kind=kind, M=_size(rng, 1, 256), N=_size(rng, 64, 8192), K=_size(rng, 64, 8192),
                    dtype=rng.choice(["f32", "f32", "f32", "bf16"]),
                    act=rng.choice(["relu", "sigmoid", "tanh", "gelu"]))
    if kind == "bmm":
        return dict(kind=kind, P=rng.randint(1, 16), Q=rng.randint(1, 8), M=_size(rng, 16, 512),
                    K=_size(rng, 16, 512), N=_size(rng, 16, 512))
    if kind == "conv":
        k = rng.choice([1, 3, 3, 5])
        # the first layer of a network reads [N][C][H][W] images of few channels
        first = rng.random() < 0.25
        H = _size(rng, 8, 56)
        return dict(kind=kind, N=rng.randint(1, 32), C=rng.choice([1, 3]) if first else rng.choice([16, 32, 48, 64, 128, 256]),
                    H=H, W=max(8, H - rng.randint(0, 3)), CO=rng.choice([20, 32, 64, 96, 128, 256]), k=k,
                    s=rng.choice([1, 1, 2]), p=k // 2, layout="nchw" if first else "cl")
    if kind == "mlp":
        return dict(kind=kind, M=_size(rng, 32, 4096), D0=_size(rng, 16, 4096), D1=_size(rng, 32, 4096),
                    D2=_size(rng, 2, 1024), act=rng.choice(["relu", "sigmoid", "tanh", "gelu"]))
    return dict(kind=kind, A=_size(rng, 2, 128), B=_size(rng, 8, 512), C=_size(rng, 8, 4096),
                keep=rng.choice(["A", "B", "C", "AB", "AC", "BC"]))


def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _uniform(g, a, *shape):
    return a * (2.0 * torch.rand(shape, generator=g, device=DEV) - 1.0)


def _out(*shape):
    return torch.empty(shape, device=DEV)


def _ws(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None


def _typed(t, c):
    return t.to(torch.bfloat16) if c.get("dtype") == "bf16" else t


def _reduced(c):
    """The shape of the un-broadcast gradient: a kept axis keeps its size."""
    return tuple(c[a] if a in c["keep"] else 1 for a in "ABC")


def _conv_out(c):
    return (c["H"] + 2 * c["p"] - c["k"]) // c["s"] + 1, (c["W"] + 2 * c["p"] - c["k"]) // c["s"] + 1


def _inputs(c, seed):
    """Activations and gradients are normal, weights and biases uniform by the layer's fan-in."""
    g, k = _gen(seed), c["kind"]
    if k == "dense" or k == "eval":
        a = 1.0 / math.sqrt(c["K"])
        d = dict(x=_typed(_normal(g, c["M"], c["K"]), c), w=_typed(_uniform(g, a, c["N"], c["K"]), c),
                 b=_uniform(g, a, c["N"]))
        if k == "dense":
            d["dy"] = _typed(_normal(g, c["M"], c["N"]), c)
        return d
    if k == "bmm":
        return dict(a=_uniform(g, 1.0, c["P"], 1, c["M"], c["K"]), b=_uniform(g, 1.0, 1, c["Q"], c["K"], c["N"]),
                    dc=_normal(g, c["P"], c["Q"], c["M"], c["N"]))
    if k == "conv":
        a = 1.0 / math.sqrt(c["C"] * c["k"] * c["k"])
        ho, wo = _conv_out(c)
        d = dict(x=_normal(g, c["N"], c["C"], c["H"], c["W"]), w=_uniform(g, a, c["CO"], c["C"], c["k"], c["k"]),
                 b=_uniform(g, a, c["CO"]), dy=_normal(g, c["N"], c["CO"], ho, wo))
        cl = torch.channels_last
        if c["layout"] == "cl":
            d["x"], d["w"] = d["x"].contiguous(memory_format=cl), d["w"].contiguous(memory_format=cl)
        d["dy"] = _cl(d["dy"])
        return d
    if k == "mlp":
        a1, a2 = 1.0 / math.sqrt(c["D0"]), 1.0 / math.sqrt(c["D1"])
        d = dict(x=_normal(g, c["M"], c["D0"]), t=_normal(g, c["M"], c["D2"]))
        d["params"] = [_uniform(g, a1, c["D1"], c["D0"]), _uniform(g, a1, c["D1"]),
                       _uniform(g, a2, c["D2"], c["D1"]), _uniform(g, a2, c["D2"])]
        d["m"] = [1e-4 * _normal(g, *p.shape) for p in d["params"]]
        d["v"] = [1e-6 * (0.5 + torch.rand(p.shape, generator=g, device=DEV)) for p in d["params"]]
        return d
    return dict(dy=_normal(g, c["A"], c["B"], c["C"]))


def _cl(t):
    """Channels-last memory whatever the sizes (a one-channel tensor's strides are ambiguous to torch)."""
    n, c, h, w = t.shape
    return t.permute(0, 2, 3, 1).contiguous().as_strided((n, c, h, w), (h * w * c, 1, w * c, c))


def prepare(case, seed):
    c = case
    st = dict(case=c, **_inputs(c, seed))
    k = c["kind"]
    if k == "dense":
        st.update(y=_out(c["M"], c["N"]), dx=_out(c["M"], c["K"]), dw=_out(c["N"], c["K"]), db=_out(c["N"]))
        st["ws"] = _ws(mt.linear_bwd_workspace(st["x"], st["w"], st["dy"], st["dx"], st["dw"], st["db"]))
    elif k == "eval":
        st["y"] = _out(c["M"], c["N"])
    elif k == "bmm":
        st.update(c=_out(c["P"], c["Q"], c["M"], c["N"]), da=torch.empty_like(st["a"]), db=torch.empty_like(st["b"]))
        # dA = sum over Q of dC B^T, dB = sum over P of A^T dC
        st.update(at=st["a"].transpose(-1, -2), bt=st["b"].transpose(-1, -2))
        n = max(mt.matmul_workspace(st["a"], st["b"], st["c"]),
                mt.matmul_workspace(st["dc"], st["bt"], st["da"], reduce_into=True),
                mt.matmul_workspace(st["at"], st["dc"], st["db"], reduce_into=True))
        st["ws"] = _ws(n)
    elif k == "conv":
        st.update(y=torch.empty_like(st["dy"]), dx=torch.empty_like(st["x"]), dw=torch.empty_like(st["w"]),
                  db=_out(c["CO"]))
        n = max(mt.conv2d_fwd_workspace(st["x"], st["w"], st["b"], st["y"], c["s"], c["p"]),
                mt.conv2d_bwd_workspace(st["x"], st["w"], st["dy"], st["dx"], st["dw"], st["db"], c["s"], c["p"]))
        st["ws"] = _ws(n)
    elif k == "mlp":
        M, D1, D2 = c["M"], c["D1"], c["D2"]
        st.update(z=_out(M, D1), h=_out(M, D1), y=_out(M, D2), loss=_out(1), dy=_out(M, D2), dh=_out(M, D1),
                  dz=_out(M, D1), grads=[torch.empty_like(p) for p in st["params"]], step=STEP)
        w1, b1, w2, b2 = st["params"]
        dw1, db1, dw2, db2 = st["grads"]
        n = max(mt.mse_loss_workspace(st["y"], st["t"]),
                mt.linear_bwd_workspace(st["h"], w2, st["dy"], st["dh"], dw2, db2),
                mt.act_bwd_workspace(c["act"], st["z"], st["dh"], st["dz"], db1),
                mt.linear_bwd_workspace(st["x"], None, st["dz"], None, dw1, None))
        st["ws"] = _ws(n)
    else:
        st["dx"] = _out(*_reduced(c))
        st["ws"] = _ws(mt.reduce_broadcast_grad_workspace(st["dy"], st["dx"]))
    return st


def run(state):
    st, c = state, state["case"]
    k = c["kind"]
    if k == "dense":
        mt.linear_fwd(st["x"], st["w"], st["b"], st["y"])
        mt.linear_bwd(st["x"], st["w"], st["dy"], st["dx"], st["dw"], st["db"], workspace=st["ws"])
        return dict(y=st["y"], dx=st["dx"], dw=st["dw"], db=st["db"])
    if k == "eval":
        mt.linear_act_fwd(st["x"], st["w"], st["b"], c["act"], st["y"])
        return dict(y=st["y"])
    if k == "bmm":
        mt.matmul(st["a"], st["b"], st["c"], workspace=st["ws"])
        mt.matmul(st["dc"], st["bt"], st["da"], reduce_into=True, workspace=st["ws"])
        mt.matmul(st["at"], st["dc"], st["db"], reduce_into=True, workspace=st["ws"])
        return dict(c=st["c"], da=st["da"], db=st["db"])
    if k == "conv":
        mt.conv2d_fwd(st["x"], st["w"], st["b"], st["y"], c["s"], c["p"], workspace=st["ws"])
        mt.conv2d_bwd(st["x"], st["w"], st["dy"], st["dx"], st["dw"], st["db"], c["s"], c["p"], workspace=st["ws"])
        return dict(y=st["y"], dx=st["dx"], dw=st["dw"], db=st["db"])
    if k == "mlp":
        w1, b1, w2, b2 = st["params"]
        dw1, db1, dw2, db2 = st["grads"]
        ws = st["ws"]
        mt.linear_act_fwd(st["x"], w1, b1, c["act"], st["h"], st["z"])
        mt.linear_fwd(st["h"], w2, b2, st["y"])
        mt.mse_loss(st["y"], st["t"], st["loss"], st["dy"], workspace=ws)
        mt.linear_bwd(st["h"], w2, st["dy"], st["dh"], dw2, db2, workspace=ws)
        mt.act_bwd(c["act"], st["z"], st["dh"], st["dz"], db1, workspace=ws)
        mt.linear_bwd(st["x"], None, st["dz"], None, dw1, None, workspace=ws)
        mt.adam_step(st["params"], st["grads"], st["m"], st["v"], LR, BETA1, BETA2, EPS, st["step"])
        st["step"] += 1
        return dict(y=st["y"], loss=st["loss"], grads=st["grads"], params=st["params"], m=st["m"], v=st["v"])
    mt.reduce_broadcast_grad(st["dy"], st["dx"], workspace=st["ws"])
    return dict(dx=st["dx"])


_ACT = dict(relu=torch.relu, sigmoid=torch.sigmoid, tanh=torch.tanh, gelu=F.gelu)


def _act_grad(act, z):
    if act == "relu":
        return (z > 0).to(z.dtype)
    if act == "sigmoid":
        s = torch.sigmoid(z)
        return s * (1 - s)
    if act == "tanh":
        return 1 - torch.tanh(z) ** 2
    return 0.5 * (1 + torch.erf(z / math.sqrt(2))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def exact(case, seed):
    c, k = case, case["kind"]
    i = _inputs(c, seed)
    d = {n: t.double() for n, t in i.items() if isinstance(t, torch.Tensor)}
    if k == "dense":
        return dict(y=d["x"] @ d["w"].t() + d["b"], dx=d["dy"] @ d["w"], dw=d["dy"].t() @ d["x"], db=d["dy"].sum(0))
    if k == "eval":
        return dict(y=_ACT[c["act"]](d["x"] @ d["w"].t() + d["b"]))
    if k == "bmm":
        out = [[d["a"][p, 0] @ d["b"][0, q] for q in range(c["Q"])] for p in range(c["P"])]
        da = [sum(d["dc"][p, q] @ d["b"][0, q].t() for q in range(c["Q"])) for p in range(c["P"])]
        db = [sum(d["a"][p, 0].t() @ d["dc"][p, q] for p in range(c["P"])) for q in range(c["Q"])]
        return dict(c=torch.stack([torch.stack(r) for r in out]), da=torch.stack(da).unsqueeze(1),
                    db=torch.stack(db).unsqueeze(0))
    if k == "conv":
        n, co, ks = c["N"], c["CO"], (c["k"], c["k"])
        ho, wo = _conv_out(c)
        wf = d["w"].reshape(co, -1)
        y, dw, dx = [], 0, []
        for b in range(n):  # an image at a time: the unfolded input in 64 bits is large
            u = F.unfold(d["x"][b:b + 1].contiguous(), ks, padding=c["p"], stride=c["s"])[0]
            g = d["dy"][b].reshape(co, -1)
            y.append((wf @ u + d["b"][:, None]).reshape(co, ho, wo))
            dw = dw + g @ u.t()
            dx.append(F.fold((wf.t() @ g)[None], (c["H"], c["W"]), ks, padding=c["p"], stride=c["s"])[0])
        like = i["dy"].stride()  # laid out as the buffers of run()
        return dict(y=_strided(torch.stack(y), like), dx=_strided(torch.stack(dx), i["x"].stride()),
                    dw=_strided(dw.reshape(d["w"].shape), i["w"].stride()), db=d["dy"].sum((0, 2, 3)))
    if k == "mlp":
        w1, b1, w2, b2 = (p.double() for p in i["params"])
        z = d["x"] @ w1.t() + b1
        h = _ACT[c["act"]](z)
        y = h @ w2.t() + b2
        loss = ((y - d["t"]) ** 2).mean().reshape(1)
        dy = 2 * (y - d["t"]) / y.numel()
        dz = (dy @ w2) * _act_grad(c["act"], z)
        grads = [dz.t() @ d["x"], dz.sum(0), dy.t() @ h, dy.sum(0)]
        lr, be1, be2, eps = _f32(LR), _f32(BETA1), _f32(BETA2), _f32(EPS)
        ms = [be1 * m.double() + (1 - be1) * g for m, g in zip(i["m"], grads)]
        vs = [be2 * v.double() + (1 - be2) * g * g for v, g in zip(i["v"], grads)]
        ps = [p.double() - lr * (m / (1 - be1 ** STEP)) / ((v / (1 - be2 ** STEP)).sqrt() + eps)
              for p, m, v in zip(i["params"], ms, vs)]
        return dict(y=y, loss=loss, grads=grads, params=ps, m=ms, v=vs)
    axes = [n for n, a in enumerate("ABC") if a not in c["keep"]]
    return dict(dx=d["dy"].sum(axes, keepdim=True))


def _strided(t, stride):
    out = torch.empty_strided(t.shape, stride, dtype=t.dtype, device=t.device)
    return out.copy_(t)


def work(case):
    c, k = case, case["kind"]
    if k == "dense" or k == "eval":
        M, N, K = c["M"], c["N"], c["K"]
        es = 2 if c["dtype"] == "bf16" else 4
        if k == "eval":
            return dict(bytes=es * (M * K + N * K) + 4 * (N + M * N), flops=2.0 * M * N * K)
        return dict(bytes=es * (M * K + N * K + M * N) + 4 * (M * N + M * K + N * K + 2 * N), flops=6.0 * M * N * K)
    if k == "bmm":
        P, Q, M, K, N = (c[n] for n in "PQMKN")
        return dict(bytes=4.0 * (2 * P * M * K + 2 * Q * K * N + 2 * P * Q * M * N), flops=6.0 * P * Q * M * N * K)
    if k == "conv":
        ho, wo = _conv_out(c)
        x, w, y = c["N"] * c["C"] * c["H"] * c["W"], c["CO"] * c["C"] * c["k"] ** 2, c["N"] * c["CO"] * ho * wo
        return dict(bytes=4.0 * (2 * x + 2 * w + 2 * y + 2 * c["CO"]),
                    flops=6.0 * c["N"] * ho * wo * c["CO"] * c["C"] * c["k"] ** 2)
    if k == "mlp":
        M, D0, D1, D2 = (c[n] for n in ("M", "D0", "D1", "D2"))
        params = D1 * D0 + D1 + D2 * D1 + D2
        # x and t read; y, the loss and the gradients written; Adam reads p, m, v and writes them
        return dict(bytes=4.0 * (M * D0 + 2 * M * D2 + 1 + 7 * params), flops=2.0 * M * (2 * D0 * D1 + 3 * D1 * D2))
    return dict(bytes=4.0 * (c["A"] * c["B"] * c["C"] + math.prod(_reduced(c))), flops=float(c["A"] * c["B"] * c["C"]))


def tolerance(case):
    # fp32 sums (products of bf16 values are exact in fp32): measured against
    # 64 bits, the path is 1e-7 off at short contractions and 1.6e-6 at 8192
    return {"rel": 1e-5}
