"""The layers a user of this package evaluates and trains, as timed cases.

Each case is one tensorial convolution layer: its conv_einsum string, sizes,
element type, and whether the pass is the forward alone (serving) or forward
plus the gradients of every operand (training).  `family` names the
factorisation, `api` the public entry point: `einsum` is the differentiable
conv_einsum() of a PyTorch program, `plan` a Plan built once whose forward /
backward the program calls each step (strided layers are only offered there).

The listed sizes are the layers the repository's benchmark, its ResNet-34
sweep and its tests name; draw() spreads over the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2401_03384_amd as P
from workloads import RESNET34_CONVS, cp_rank

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_SPECS = {
    "cp": "bshw,rs,rt,rh,rw->bthw|hw",
    "tucker": "bshw,sp,pqhw,qt->bthw|hw",
    "rtt": ("b(s1)(s2)(s3)hw,(r1)(t1)(s1),(r1)(r2)(t2)(s2),(r2)(r3)(t3)(s3),(r3)hw"
            "->b(t1)(t2)(t3)hw|hw"),
    "rcp": "b(s1)(s2)(s3)hw,r(t1)(s1),r(t2)(s2),r(t3)(s3),rhw->b(t1)(t2)(t3)hw|hw",
}


def _cp(b, s, t, h, w, r, k, dtype, train=True, api="plan", stride=1, **kw):
    return dict(kw, family="cp", b=b, s=s, t=t, h=h, w=w, r=r, k=k, stride=stride, dtype=dtype,
                train=train, api=api)


def _tucker(b, s, t, h, w, p, q, k, dtype, train=True, api="plan", **kw):
    return dict(kw, family="tucker", b=b, s=s, t=t, h=h, w=w, p=p, q=q, k=k, stride=1,
                dtype=dtype, train=train, api=api)


def _reshaped(family, b, ss, ts, h, w, r, k, dtype, train=True, api="plan", **kw):
    return dict(kw, family=family, b=b, s1=ss[0], s2=ss[1], s3=ss[2], t1=ts[0], t2=ts[1],
                t3=ts[2], h=h, w=w, r=r, k=k, stride=1, dtype=dtype, train=train, api=api)


def _resnet(conv, b, dtype, train=True, **kw):
    """A ResNet-34 convolution as a CP layer holding the dense kernel's
    parameter count (compression rate 100%)."""
    _, s, t, hw, k, st = {r[0]: r for r in RESNET34_CONVS}[conv]
    return _cp(b, s, t, hw, hw, cp_rank(s, t, k), k, dtype, train, stride=st, **kw)


def listed():
    return [
        # the smallest call: an 8x8 CP layer in a PyTorch program (latency)
        _cp(2, 16, 16, 8, 8, 8, 3, "f32", api="einsum", name="cp_tiny_f32"),
        # serving one image through a ResNet stage-1 sized CP layer
        _cp(1, 64, 64, 56, 56, 32, 3, "bf16", train=False, name="cp_serve_bf16"),
        # the benchmark's headline layer: ResNet stage 1, rank 32, batch 128
        _cp(128, 64, 64, 56, 56, 32, 3, "f32", api="einsum", name="cp_stage1_f32"),
        _cp(128, 64, 64, 56, 56, 32, 3, "bf16", name="cp_stage1_bf16"),
        # channel counts, planes and rank off the round numbers, 5x5 taps
        _cp(24, 48, 40, 37, 29, 20, 5, "f32", name="cp_ragged_k5_f32"),
        # Tucker-2 training at a ResNet stage-3 shape
        _tucker(128, 256, 256, 14, 14, 64, 64, 3, "bf16", name="tucker_stage3_bf16"),
        # evaluating a Tucker-2 layer with ragged planes and ranks
        _tucker(16, 96, 72, 13, 27, 40, 48, 3, "f32", train=False, api="einsum",
                name="tucker_ragged_f32"),
        # reshaped tensor-train training, 256 channels, 28x28
        _reshaped("rtt", 64, (4, 8, 8), (4, 8, 8), 28, 28, 16, 3, "f32", name="rtt_28x28_f32"),
        # reshaped CP training: 512 channels on 7x7, 128 channels on 28x28 (5x5)
        _reshaped("rcp", 32, (8, 8, 8), (8, 8, 8), 7, 7, 64, 3, "bf16", name="rcp_7x7_bf16"),
        _reshaped("rcp", 32, (4, 4, 8), (4, 4, 8), 28, 28, 64, 5, "bf16", name="rcp_28x28_k5_bf16"),
        # ResNet-34 layers at the dense kernel's parameter count: a repeated
        # 3x3 and a stage-entry stride-2 one
        _resnet("conv3_x", 16, "f32", name="resnet_conv3_f32"),
        _resnet("conv4_1", 16, "bf16", name="resnet_conv4_s2_bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more layer of the same ranges: any family, both element types,
    training or evaluation, sizes over the whole range."""
    limit = max(work(c)["flops"] for c in listed())
    family = rng.choice(["cp", "cp", "resnet", "tucker", "rtt", "rcp", "rcp"])
    dtype = rng.choice(["f32", "bf16"])
    train = rng.random() < 0.75
    h = _log_int(rng, 7, 56)
    w = h if rng.random() < 0.5 else _log_int(rng, 7, 56)
    k = rng.choice([3, 3, 5])
    if family == "resnet":
        c = _resnet(rng.choice(RESNET34_CONVS)[0], _log_int(rng, 1, 16), dtype, train)
    elif family == "cp":
        c = _cp(_log_int(rng, 1, 128), rng.randint(16, 64), rng.randint(16, 64), h, w,
                rng.randint(8, 32), k, dtype, train)
    elif family == "tucker":
        c = _tucker(_log_int(rng, 1, 128), _log_int(rng, 16, 256), _log_int(rng, 16, 256),
                    min(h, 28), min(w, 28), rng.randint(8, 64), rng.randint(8, 64), k, dtype, train)
    else:
        modes = [(4, 8, 8), (8, 8, 8), (4, 4, 8), (4, 4, 4), (2, 4, 8), (3, 5, 6)]
        ss = rng.choice(modes)
        ts = ss if rng.random() < 0.7 else rng.choice(modes)
        r = rng.randint(4, 16) if family == "rtt" else _log_int(rng, 4, 64)
        c = _reshaped(family, _log_int(rng, 1, 64), ss, ts, min(h, 28), min(w, 28), r,
                      3 if family == "rtt" else k, dtype, train)
    if c["stride"] == 1 and rng.random() < 0.4:
        c["api"] = "einsum"
    while c["b"] > 1 and work(c)["flops"] > limit:
        c["b"] //= 2
    return c


def _shapes(c):
    b, h, w, k = c["b"], c["h"], c["w"], c["k"]
    if c["family"] == "cp":
        s, t, r = c["s"], c["t"], c["r"]
        return [(b, s, h, w), (r, s), (r, t), (r, k), (r, k)]
    if c["family"] == "tucker":
        s, t, p, q = c["s"], c["t"], c["p"], c["q"]
        return [(b, s, h, w), (s, p), (p, q, k, k), (q, t)]
    ss, ts, r = [c["s1"], c["s2"], c["s3"]], [c["t1"], c["t2"], c["t3"]], c["r"]
    x = (b, *ss, h, w)
    if c["family"] == "rtt":
        return [x, (r, ts[0], ss[0]), (r, r, ts[1], ss[1]), (r, r, ts[2], ss[2]), (r, k, k)]
    return [x, (r, ts[0], ss[0]), (r, ts[1], ss[1]), (r, ts[2], ss[2]), (r, k, k)]


def _sigmas(c):
    """Standard deviations: N(0, 1) features; factors such that the dense
    kernel they stand for has variance 2 / fan_in (Kaiming)."""
    if c["family"] == "cp":
        fan, ranks, n = c["s"], c["r"], 4
    elif c["family"] == "tucker":
        fan, ranks, n = c["s"], c["p"] * c["q"], 3
    else:
        fan, n = c["s1"] * c["s2"] * c["s3"], 4
        ranks = c["r"] ** (3 if c["family"] == "rtt" else 1)
    sg = (2.0 / (fan * c["k"] ** 2 * ranks)) ** (1.0 / (2 * n))
    return [1.0] + [sg] * n


def _plan(c):
    strides = {"h": c["stride"], "w": c["stride"]} if c["stride"] > 1 else None
    return P.Plan(_SPECS[c["family"]], _shapes(c), c["dtype"], strides=strides)


def _inputs(c, seed, device):
    """Operands and output gradient, drawn from the seed alone."""
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    dt = _TORCH[c["dtype"]]
    xs = [(torch.randn(s, generator=g, device=device) * sg).to(dt)
          for s, sg in zip(_shapes(c), _sigmas(c))]
    h, w = -(-c["h"] // c["stride"]), -(-c["w"] // c["stride"])
    ts = [c["t"]] if c["family"] in ("cp", "tucker") else [c["t1"], c["t2"], c["t3"]]
    dy = torch.randn((c["b"], *ts, h, w), generator=g, device=device).to(dt)
    return xs, dy


def prepare(case, seed):
    xs, dy = _inputs(case, seed, torch.device("cuda"))
    state = {"xs": xs, "dy": dy, "train": case["train"], "spec": _SPECS[case["family"]]}
    if case["api"] == "plan":
        state["plan"] = _plan(case)
    elif case["train"]:
        state["xs"] = [x.requires_grad_() for x in xs]
    return state


def run(state):
    xs = state["xs"]
    if "plan" in state:
        y = state["plan"].forward(xs)
        return [y, *state["plan"].backward(xs, state["dy"])] if state["train"] else [y]
    y = P.conv_einsum(state["spec"], *xs)
    return [y, *torch.autograd.grad(y, xs, state["dy"])] if state["train"] else [y]


def work(case):
    """Multiply-adds of the cheapest pairwise order (three times the
    forward's for training); operands, output, output gradient and gradients
    moved once."""
    p = _plan(case)
    e = 2 if case["dtype"] == "bf16" else 4
    nx, ny = math.prod(p.shapes[0]), math.prod(p.out_shape)
    nf = sum(math.prod(s) for s in p.shapes[1:])
    if not case["train"]:
        return {"bytes": e * (nx + ny + nf), "flops": 2 * p.fwd_macs}
    return {"bytes": e * (2 * nx + 2 * ny + nf) + (4 if case["api"] == "plan" else e) * nf,
            "flops": 6 * p.fwd_macs}


def tolerance(case):
    """Four times the largest distance from the 64-bit result that the listed
    layers show: fp32 sums (1.2e-6), or bf16 operands, intermediates and
    results with fp32 sums (3.3e-3)."""
    return {"rel": 1.4e-2} if case["dtype"] == "bf16" else {"rel": 5e-6}


def _kernel(family, f):
    """The dense kernel [t, s, kh, kw] that a layer's factors stand for."""
    if family == "cp":
        a = f[0][:, :, None, None] * f[2][:, None, :, None] * f[3][:, None, None, :]
        return torch.einsum("rt,rz->tz", f[1], a.flatten(1)).reshape(-1, *a.shape[1:])
    if family == "tucker":
        return torch.einsum("sp,ptz->tsz", f[0],
                            torch.einsum("pqz,qt->ptz", f[1].flatten(2), f[2])
                            ).unflatten(2, f[1].shape[2:])
    if family == "rcp":
        a = torch.einsum("rax,rby->rabxy", f[0], f[1])
        b = torch.einsum("rcz,rk->rczk", f[2], f[3].flatten(1))
        d = torch.einsum("ru,rv->uv", a.flatten(1), b.flatten(1))
        d = d.reshape(*a.shape[1:], *b.shape[1:])                       # a b x y c z k
    else:
        a = torch.einsum("max,mnby->nabxy", f[0], f[1])
        b = torch.einsum("nocz,ok->nczk", f[2], f[3].flatten(1))
        d = torch.einsum("nu,nv->uv", a.flatten(1), b.flatten(1))
        d = d.reshape(*a.shape[1:], *b.shape[1:])
    d = d.permute(0, 1, 4, 2, 3, 5, 6)                                   # a b c x y z k
    return d.reshape(math.prod(d.shape[:3]), math.prod(d.shape[3:6]), *f[3].shape[1:])


def exact(case, seed):
    """The dense convolution, its chain rule and the merged factors' chain
    rule in float64."""
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    xs, dy = _inputs(case, seed, device)
    x = xs[0].double().flatten(1, -3)
    fs = [v.double().requires_grad_() for v in xs[1:]]
    k, st, (ho, wo) = case["k"], case["stride"], dy.shape[-2:]
    lo, (b, s, h, w) = (k - 1) // 2, x.shape
    pad = torch.zeros(s, b, h + k - 1, w + k - 1, dtype=x.dtype, device=device)
    pad[:, :, lo:lo + h, lo:lo + w] = x.transpose(0, 1)
    kernel = _kernel(case["family"], fs)
    kd = kernel.detach()
    t = kd.shape[0]
    taps = [(i, j) for i in range(k) for j in range(k)]

    def view(a, i, j):
        return a[:, :, i:i + st * (ho - 1) + 1:st, j:j + st * (wo - 1) + 1:st]

    y = torch.zeros(t, b * ho * wo, dtype=x.dtype, device=device)
    for i, j in taps:
        y += kd[:, :, i, j].contiguous() @ view(pad, i, j).reshape(s, -1)
    y = y.reshape(t, b, ho, wo).transpose(0, 1).reshape(dy.shape)
    if not case["train"]:
        return [y]
    d = dy.double().flatten(1, -3).transpose(0, 1).reshape(t, -1)
    dpad, dk = torch.zeros_like(pad), torch.zeros_like(kd)
    for i, j in taps:
        dk[:, :, i, j] = d @ view(pad, i, j).reshape(s, -1).T
        view(dpad, i, j).add_((kd[:, :, i, j].T.contiguous() @ d).reshape(s, b, ho, wo))
    dx = dpad[:, :, lo:lo + h, lo:lo + w].transpose(0, 1).reshape(xs[0].shape)
    return [y, dx, *torch.autograd.grad(kernel, fs, dk)]
