"""The work that the hot path's figures are measured on.

A case is one layer-step (or one other call a training program makes) at one size.  `listed()` gives the fixed ones,
`draw()` more of the same ranges; `prepare` makes what a training program holds before the call, `run` is one pass
through the public entry points, `work` and `tolerance` say what the pass cannot do without and how closely two
correct implementations agree.

Kinds of a case:
  step      LayerRunner.step: asi_compress, asi_core_project and asi_weight_grad_* of one layer, warm-started
  batch     BatchRunner.step: the same for `count` layers of one shape through the batched entry points
  autograd  AsiLinear forward and backward: the framework's own products beside the compressed weight gradient
  ranks     perplexity_row: one layer's row of the rank-selection tables (made once per layer before training)
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2505_05086_amd import binding as B
from paper_2505_05086_amd.autograd import AsiLinear
from paper_2505_05086_amd.rank_selection import perplexity_row
from paper_2505_05086_amd.runner import BatchRunner, LayerRunner


def _conv(name, dims, ranks, cout, k=3, stride=1, groups=1, dtype="f32", alpha=1.5, kind="step", count=1):
    case = dict(kind=kind, layer="conv2d", b=dims[0], c=dims[1], h=dims[2], w=dims[3], r1=ranks[0], r2=ranks[1],
                r3=ranks[2], r4=ranks[3], cout=cout, k=k, stride=stride, groups=groups, dtype=dtype, alpha=alpha,
                count=count)
    return dict(case, name=name) if name else case


def _linear(name, dims, ranks, cout, dtype="bf16", alpha=1.2, kind="step", count=1):
    case = dict(kind=kind, layer="linear", b=dims[0], n=dims[1], d=dims[2], r1=ranks[0], r2=ranks[1], r3=ranks[2],
                cout=cout, dtype=dtype, alpha=alpha, count=count)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a small 3x3 layer at batch 8: a microcontroller-sized model, where launches and latency count
        _conv("conv-small", (8, 32, 16, 16), (4, 8, 6, 6), 32),
        # last-stage input of a residual network at batch 64
        _conv("conv-14x14", (64, 256, 14, 14), (16, 32, 7, 7), 256),
        # its three equal 7x7 layers, stepped together
        _conv("conv-7x7-batch", (64, 512, 7, 7), (16, 48, 5, 5), 512, kind="batch", count=3),
        # mobile network tail at batch 128: depthwise 3x3 and the pointwise projection after it
        _conv("conv-depthwise", (128, 960, 7, 7), (24, 40, 6, 6), 960, groups=960),
        _conv("conv-pointwise", (128, 960, 7, 7), (24, 40, 6, 6), 320, k=1),
        # segmentation-sized maps; the second has the batch mode at full rank
        _conv("conv-56x56", (32, 128, 56, 56), (16, 32, 24, 24), 128, alpha=1.0),
        _conv("conv-64x64", (8, 256, 64, 64), (8, 48, 32, 32), 256, alpha=1.0),
        # nothing divides anything: odd batch, channels, maps and ranks, stride 2
        _conv("conv-ragged", (13, 83, 45, 37), (9, 21, 15, 13), 101, stride=2),
        # second linear layer of a vision transformer's feed-forward block, the largest rank
        _linear("linear-vit-fc2", (64, 197, 3072), (32, 64, 192), 768),
        # widest linear layer of a language model's decoder block: tiny ranks, full-rank batch mode
        _linear("linear-llm-up", (8, 512, 2048), (8, 20, 20), 5632),
        # an attention projection of the same block in a training loop: forward and backward through autograd
        _linear("autograd-llm-attn", (8, 512, 2048), (8, 20, 20), 2048, kind="autograd"),
        # choosing the ranks of a pointwise layer before training
        _conv("ranks-pointwise", (128, 160, 7, 7), (24, 40, 6, 6), 960, k=1, kind="ranks"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more layer: mostly single layer-steps, sizes over the whole range of the listed ones."""
    kind = rng.choice(["step"] * 8 + ["batch", "autograd"])
    conv = kind == "batch" or (kind == "step" and rng.random() < 0.65)
    while True:
        if conv:
            b, c, h = _log(rng, 4, 128), _log(rng, 16, 1024), _log(rng, 7, 64)
            w = h if rng.random() < 0.7 else max(4, min(64, h + rng.randint(-5, 5)))
            if not 2.5e5 <= b * c * h * w <= 1.3e7:
                continue
            if rng.random() < 0.6:                       # widths that networks have
                b, c = max(4, b // 8 * 8), max(16, c // 16 * 16)
            ranks = (max(2, min(b, 32, int(b * rng.choice([0.19, 0.25, 0.5, 1.0])))), max(4, min(64, int(c * rng.uniform(0.05, 0.25)))),
                     max(2, min(32, int(h * rng.uniform(0.4, 0.9)))), max(2, min(32, int(w * rng.uniform(0.4, 0.9)))))
            k, groups = rng.choice([(1, 1), (1, 1), (3, 1), (3, 1), (3, 1), (3, c), (5, 1)])
            stride = 2 if rng.random() < 0.15 else 1
            cout = c if groups > 1 else max(16, min(1280, int(c * rng.choice([0.5, 1, 1, 1, 2, 3]))))
            case = _conv(None, (b, c, h, w), ranks, cout, k, stride, groups, rng.choice(["f32"] * 4 + ["bf16"]),
                         rng.choice([1.0, 1.5]), kind, rng.randint(2, 4) if kind == "batch" and b * c * h * w < 4e6 else
                         2 if kind == "batch" else 1)
            if _sensible(case):
                return case
            continue
        b, n, d = _log(rng, 4, 64), _log(rng, 49, 512), _log(rng, 192, 5632)
        if not 5e5 <= b * n * d <= 3.8e7:
            continue
        if rng.random() < 0.6:
            d = d // 64 * 64
        ranks = (max(2, int(b * rng.choice([0.5, 1.0]))), max(8, min(64, int(n * rng.uniform(0.04, 0.33)))),
                 max(8, min(192, int(d * rng.uniform(0.01, 0.125)))))
        cout = max(192, min(5632, int(d * rng.choice([0.25, 1, 1, 1, 2.75, 4]))))
        case = _linear(None, (b, n, d), ranks, cout, rng.choice(["bf16", "bf16", "f32"]), 1.2, kind)
        if _sensible(case):
            return case


def _sensible(case):
    """No mode asks for more directions than the others can tell apart, and nothing costs more than the listed layers."""
    ranks = [case[k] for k in ("r1", "r2", "r3", "r4") if k in case]
    w = work(case)
    return all(2 * r * r <= _prod(ranks) for r in ranks) and w["bytes"] <= 1.1e8 and w["flops"] <= 5.4e10


# ---- sizes ----------------------------------------------------------------------------------------------------
def _layer(case):
    if case["layer"] == "conv2d":
        dims = (case["b"], case["c"], case["h"], case["w"])
        ranks = (case["r1"], case["r2"], case["r3"], case["r4"])
        k, pad = case["k"], (case["k"] - 1) // 2
        ho, wo = ((x + 2 * pad - k) // case["stride"] + 1 for x in dims[2:])
        gy = (dims[0], case["cout"], ho, wo)
        dw = (case["cout"], dims[1] // case["groups"], k, k)
        return SimpleNamespace(dims=dims, ranks=ranks, dtype=case["dtype"], kind="conv2d", cout=case["cout"], k=k,
                               stride=case["stride"], pad=pad, dil=1, groups=case["groups"], grad_out_shape=gy, dw_shape=dw)
    dims, ranks = (case["b"], case["n"], case["d"]), (case["r1"], case["r2"], case["r3"])
    return SimpleNamespace(dims=dims, ranks=ranks, dtype=case["dtype"], kind="linear", cout=case["cout"], k=1, stride=1,
                           pad=0, dil=1, groups=1, grad_out_shape=(dims[0], dims[1], case["cout"]),
                           dw_shape=(case["cout"], dims[2]))


# ---- inputs -----------------------------------------------------------------------------------------------------
_NOISE, _DRIFT = 1e-3, 0.02      # noise beside a signal of unit RMS; how far the factors move in one training step


def _orthonormal(x):
    q, r = np.linalg.qr(x)
    return q * np.sign(np.diag(r))


def _inputs(lay, alpha, seed):
    """(activation, grad_out, factors of the previous step) of one layer: a Tucker tensor whose singular values decay
    as i^-alpha in every mode, plus noise; the factors a warm-started run holds, i.e. the leading singular vectors of
    an activation that has drifted a little since."""
    rng = np.random.default_rng(seed)
    core = rng.standard_normal(lay.ranks)
    for m, r in enumerate(lay.ranks):
        core *= (np.arange(1, r + 1.0) ** -alpha).reshape([-1 if q == m else 1 for q in range(len(lay.ranks))])
    factors, previous = [], []
    for m, (n, r) in enumerate(zip(lay.dims, lay.ranks)):
        f = _orthonormal(rng.standard_normal((n, r)))
        u = np.moveaxis(core, m, 0).reshape(r, -1)
        vec = np.linalg.eigh(u @ u.T)[1][:, ::-1]
        factors.append(f)
        previous.append(_orthonormal(f @ vec + _DRIFT / math.sqrt(n) * rng.standard_normal((n, r))))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.from_numpy(core.astype(np.float32)).cuda()
    for f in factors:            # every product turns its mode to the end, so the modes come back in order
        x = torch.tensordot(x, torch.from_numpy(np.ascontiguousarray(f.T, dtype=np.float32)).cuda(), dims=([0], [0]))
    x /= x.square().mean().sqrt()
    x += _NOISE * torch.randn(lay.dims, device="cuda", generator=gen)
    gy = torch.randn(lay.grad_out_shape, device="cuda", generator=gen)
    dt = torch.float32 if lay.dtype == "f32" else torch.bfloat16
    return x.to(dt).contiguous(), gy.to(dt).contiguous(), previous


def prepare(case, seed):
    lay, kind = _layer(case), case["kind"]
    if kind == "step":
        run_ = LayerRunner(lay)
        x, gy, u = _inputs(lay, case["alpha"], seed)
        run_.set_factors(u)
        return dict(kind=kind, runner=run_, x=x, gy=gy)
    if kind == "batch":
        runner, xs, gys = BatchRunner([lay] * case["count"]), [], []
        for i, r in enumerate(runner.runs):
            x, gy, u = _inputs(lay, case["alpha"], seed + 1000003 * i)
            r.set_factors(u)
            xs.append(x)
            gys.append(gy)
        return dict(kind=kind, runner=runner, x=xs, gy=gys)
    x, gy, _ = _inputs(lay, case["alpha"], seed)
    if kind == "autograd":
        torch.manual_seed(seed)
        layer = AsiLinear(lay.dims[2], lay.cout, ranks=lay.ranks, seed=seed, device="cuda", dtype=x.dtype)
        for _ in range(4):       # past the cold start, as a training run is for all but its first steps
            layer(x)
        return dict(kind=kind, layer=layer, x=x.requires_grad_(), gy=gy)
    # ranks: the exact gradient of a pointwise convolution, as the framework's backward pass would deliver it
    exact = gy.float().transpose(0, 1).reshape(lay.cout, -1) @ x.float().transpose(0, 1).reshape(lay.dims[1], -1).t()
    conv = B.make_conv(lay.cout, 1, 1)
    return dict(kind=kind, x=x, gy=gy, exact=exact.reshape(lay.dw_shape).contiguous(), conv=conv)


def run(state):
    kind = state["kind"]
    if kind == "step":
        runner = state["runner"]
        dw = runner.step(state["x"], state["gy"])
        return dict(U=runner.factors(), S=runner.S, dW=dw)
    if kind == "batch":
        runner = state["runner"]
        dw = runner.step(state["x"], state["gy"])
        return dict(U=[r.factors() for r in runner.runs], S=[r.S for r in runner.runs], dW=dw)
    if kind == "autograd":
        layer, x = state["layer"], state["x"]
        y = layer(x)
        gx, gw, gb = torch.autograd.grad(y, (x, layer.weight, layer.bias), state["gy"])
        return dict(y=y, gx=gx, gw=gw, gb=gb, U=layer.asi.U_prev)
    t = perplexity_row(state["x"], state["gy"], state["exact"], conv=state["conv"])
    return dict(ranks=[list(r) for r in t.ranks], memory=t.memory, perplexity=t.perplexity)


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def _prod(v):
    return math.prod(int(x) for x in v)


def _core_macs(dims, ranks):
    """Cheapest chain of mode products."""
    best = [None]

    def go(cur, left, spent):
        if best[0] is not None and spent >= best[0]:
            return
        if not left:
            best[0] = spent
            return
        size = _prod(cur)
        for m in left:
            go(cur[:m] + [ranks[m]] + cur[m + 1:], [q for q in left if q != m], spent + size * ranks[m])

    go(list(dims), list(range(len(dims))), 0)
    return best[0]


def work(case):
    lay = _layer(case)
    es = 4 if lay.dtype == "f32" else 2
    numel, gyn, dwn = _prod(lay.dims), _prod(lay.grad_out_shape), _prod(lay.dw_shape)
    pack = _prod(lay.ranks) + sum(n * r for n, r in zip(lay.dims, lay.ranks))
    if case["kind"] == "ranks":
        gram = sum(numel * n for n in lay.dims)                        # half of 2 numel n: the matrix is symmetric
        return dict(bytes=es * (numel + gyn) + 4 * dwn, flops=gram + sum(9 * n ** 3 for n in lay.dims))
    r = lay.ranks
    macs = sum(2 * numel * q for q in r) + _core_macs(lay.dims, r)
    if lay.kind == "conv2d":
        g1 = r[0] * gyn
        z = r[0] * r[1] * (r[2] * r[3] * lay.dims[2] + r[3] * lay.dims[2] * lay.dims[3])
        t = r[0] * r[1] * gyn // lay.dims[0] * lay.k ** 2
        macs += g1 + z + t + r[1] * dwn
    else:
        macs += r[0] * gyn + r[0] * r[1] * lay.dims[1] * lay.cout + r[0] * r[1] * r[2] * lay.cout + r[2] * dwn
    nbytes = es * (numel + gyn) + 4 * (dwn + pack + sum(n * q for n, q in zip(lay.dims, r)))
    if case["kind"] == "autograd":
        macs += 2 * _prod(lay.dims) * lay.cout                          # y = x W^T and dx = dy W
        nbytes = es * (2 * numel + 2 * gyn + 2 * dwn) + 8 * sum(n * q for n, q in zip(lay.dims, r))
    return dict(bytes=case["count"] * nbytes, flops=2 * case["count"] * macs)


def tolerance(case):
    # Measured against the same step in float64, over the listed and a dozen drawn layers: the largest relative error
    # of an output is 2.8e-6 for fp32 inputs (channel factor of a layer whose singular values span three decades) and
    # 8.9e-6 for bf16 inputs (192 directions of a 3072-long mode), the largest single error 4.3e-5 and 3.4e-4 of the
    # output's rms.  About four times that.  Autograd layers round dW, dx and y to the weight's type.
    if case["kind"] == "autograd":
        return {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 1e-4, "max": 2e-3}
    return {"rel": 4e-5, "max": 1.5e-3} if case["dtype"] == "bf16" else {"rel": 1.2e-5, "max": 2e-4}
