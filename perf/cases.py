"""Measured cases of the Jorge optimizer step, through the Python entry points.

A case is one context (a list of m x n layers) and one way of stepping it:

* entry "step":      Jorge.step, tensors handed over and checked on every call;
* entry "ptrs":      Jorge.step_ptrs, for a program that keeps its parameter and
                     gradient buffers and so the pointer arrays to them;
* entry "optimizer": JorgeOptimizer.step, the torch.optim front end, with the
                     vector parameters (biases, normalisation scales) of a model;
* entry "noalloc":   Jorge.step_noalloc, one layer whose state the caller holds.

"update" says whether the pass updates the factors (every step of a run with
update interval 1, one in k otherwise) or is a step between two updates.

prepare() restores a mid-training state (as from a checkpoint): factors of the
size at which the update is stationary, (k sigma^2)^(-1/4) for a statistic of
rank k, with a random symmetric part that does not commute with the gradient's;
momenta of the size ten steps leave. Updating passes go through a cycle of
gradients, since one gradient repeated for thousands of steps would leave
directions that no step ever sees. The gradients of a cycle are windows of one
random buffer.
"""
from __future__ import annotations

import math

import torch

from paper_2310_12298_amd.jorge import Jorge
from paper_2310_12298_amd.optim import JorgeOptimizer
from paper_2310_12298_amd.workloads import many_small_shapes, resnet50_weight_shapes

HYPER = dict(lr=0.1, beta2=0.9, beta1=0.9, weight_decay=5e-5)
NO_UPDATE = 1 << 30        # an update interval that the passes of a run never reach
ALIGN = 64                 # floats: every tensor of a flat buffer starts 256-byte aligned
SHOWN = 14                 # layers whose whole state a pass returns (all of a smaller context)


def listed():
    return [
        # The smallest call: one 64 -> 64 3x3 convolution (ResNet-50's first stage). Launches and latency.
        {"name": "conv_64x576", "net": "one", "rows": 64, "cols": 576, "sigma": 1e-2, "entry": "step", "update": True},
        # One large convolution: 512 -> 512 3x3, the widest of ResNet-50. One explicit and one factored factor.
        {"name": "conv_512x4608", "net": "one", "rows": 512, "cols": 4608, "sigma": 1e-3, "entry": "step",
         "update": True},
        # A language model's output head or embedding slice: tall and thin, low-rank factor of 8192.
        {"name": "head_8192x512", "net": "one", "rows": 8192, "cols": 512, "sigma": 1e-3, "entry": "step",
         "update": True},
        # Every weight matrix of ResNet-50 with a factor update: the framework's headline workload.
        {"name": "resnet50_update", "net": "resnet50", "sigma": 1e-3, "entry": "ptrs", "update": True},
        # The same model through torch.optim between two updates: 49 of 50 steps at the paper's interval.
        {"name": "resnet50_between", "net": "resnet50", "sigma": 1e-3, "entry": "optimizer", "update": False},
        # A model of large dense layers (the MLP and attention matrices of a transformer), the largest case.
        {"name": "large_dense", "net": "dense", "layers": 8, "width": 4096, "narrow": 1024, "sigma": 1e-3,
         "entry": "ptrs", "update": True},
        # Hundreds of small layers of mixed sizes: short products, many per launch.
        {"name": "many_small", "net": "many_small", "layers": 512, "seed": 0, "sigma": 1e-2, "entry": "ptrs",
         "update": True},
        # The same layers between updates.
        {"name": "many_small_between", "net": "many_small", "layers": 512, "seed": 0, "sigma": 1e-2,
         "entry": "ptrs", "update": False},
        # Adapter-sized matrices only: the path that keeps a whole factor update in LDS.
        {"name": "adapters_128", "net": "equal", "layers": 256, "rows": 128, "cols": 128, "sigma": 1e-2,
         "entry": "ptrs", "update": True},
        # A few tiny layers (a small head or control network).
        {"name": "tiny_8", "net": "ragged", "layers": 8, "low": 17, "high": 64, "seed": 3, "sigma": 1e-2,
         "entry": "step", "update": True},
        # Sizes that are no multiple of anything, narrow to wide, through torch.optim.
        {"name": "ragged_24", "net": "ragged", "layers": 24, "low": 33, "high": 2100, "seed": 5, "sigma": 1e-3,
         "entry": "optimizer", "update": True},
        # A caller that may not allocate: one layer, its state in the caller's tensors.
        {"name": "noalloc_256x1024", "net": "one", "rows": 256, "cols": 1024, "sigma": 1e-3, "entry": "noalloc",
         "update": True},
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _side(rng, low, high):
    """A layer's side: log-uniform; a multiple of 64 or of 8, or any number."""
    v = _log_int(rng, low, high)
    step = rng.choice((64, 8, 1))
    return max(low, min(high, (v + step // 2) // step * step)) if step > 1 else v


def draw(rng):
    """A case of the same ranges: one layer up to 8192 wide, or a net of up to 512 layers."""
    limit = work(next(c for c in listed() if c["name"] == "large_dense"))["flops"]
    while True:
        kind = rng.choice(("one", "one", "equal", "ragged", "ragged", "many_small"))
        sigma = rng.choice((1e-2, 1e-3))
        update = rng.random() < 0.75
        entry = rng.choice(("step", "ptrs", "optimizer"))
        if kind == "one":
            case = {"net": "one", "rows": _side(rng, 16, 8192), "cols": _side(rng, 16, 8192)}
            if max(case["rows"], case["cols"]) <= 768 and rng.random() < 0.4:
                entry = "noalloc"
        elif kind == "equal":
            case = {"net": "equal", "layers": _log_int(rng, 4, 256), "rows": _side(rng, 32, 1024),
                    "cols": _side(rng, 32, 4096)}
        elif kind == "ragged":
            low, high = _log_int(rng, 16, 64), _log_int(rng, 64, 4096)
            case = {"net": "ragged", "layers": _log_int(rng, 4, 64), "low": low, "high": max(high, 2 * low),
                    "seed": rng.randrange(1 << 16)}
        else:
            case = {"net": "many_small", "layers": _log_int(rng, 16, 512), "seed": rng.randrange(1 << 16)}
        case.update(sigma=sigma, entry=entry, update=update)
        w = work(case)
        if w["flops"] <= limit and w["bytes"] <= 8e9:
            return case


def shapes_of(case):
    net = case["net"]
    if net == "one":
        return [(case["rows"], case["cols"])]
    if net == "equal":
        return [(case["rows"], case["cols"])] * case["layers"]
    if net == "resnet50":
        return resnet50_weight_shapes()
    if net == "many_small":
        return many_small_shapes(case["layers"], case["seed"])
    if net == "dense":
        return [(case["width"], case["width"])] * case["layers"] + [(case["width"], case["narrow"])] * case["layers"]
    gen = torch.Generator().manual_seed(case["seed"])
    span = math.log(case["high"] / case["low"])
    u = torch.rand(case["layers"], 2, generator=gen).tolist()
    return [tuple(int(case["low"] * math.exp(span * x)) for x in p) for p in u]


def vectors_of(case):
    """Vector parameters of a model stepped through torch.optim: two per layer (a normalisation's scale and shift)."""
    return [m for m, _ in shapes_of(case) for _ in range(2)] if case["entry"] == "optimizer" else []


# ------------------------------------------------------------------ inputs

def _offsets(sizes):
    """Start of each tensor in a flat buffer, and the buffer's length."""
    at, out = 0, []
    for n in sizes:
        out.append(at)
        at += -(-n // ALIGN) * ALIGN
    return out, at


def _cycle(case):
    """Gradients in a cycle: enough that their rows and columns span every layer's sides."""
    if not case["update"]:
        return 1
    ratio = max(max(m, n) / min(m, n) for m, n in shapes_of(case))
    return min(96, 4 + 2 * math.ceil(ratio))


def _shift(i):
    """Start of the i-th gradient's window in the random buffer."""
    return i * 37 * ALIGN


def _inputs(case, seed):
    """Everything a pass reads, as device tensors made from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def randn(*size):
        return torch.randn(*size, generator=gen, device="cuda", dtype=torch.float32)

    shapes, sigma = shapes_of(case), case["sigma"]
    offs, total = _offsets([m * n for m, n in shapes])
    theta = torch.zeros(total, device="cuda")
    moms, msgds, factors = [], [], []
    for (m, n), o in zip(shapes, offs):
        theta[o:o + m * n] = randn(m * n) * math.sqrt(2.0 / n)
        pair = []
        for d, k in ((m, n), (n, m)):
            s = randn(d, d)
            a = (s + s.t()) * (0.25 / math.sqrt(2.0 * d))
            a.diagonal().add_(1.0)
            pair.append(a.mul_((k * sigma * sigma) ** -0.25).contiguous())
        factors.append(pair)
        moms.append(randn(m, n) * (0.3 * sigma * (m * n * sigma ** 4) ** -0.25))
        msgds.append(randn(m, n) * (2.0 * sigma))
    noise = randn(total + _shift(_cycle(case))) * sigma
    voffs, vtotal = _offsets(vectors_of(case))
    vec = torch.zeros(max(vtotal, 1), device="cuda")
    vec_mom, vec_grad = randn(max(vtotal, 1)) * (2.0 * sigma), randn(max(vtotal, 1)) * sigma
    return dict(shapes=shapes, offs=offs, theta=theta, moms=moms, msgds=msgds, factors=factors, noise=noise,
                voffs=voffs, vec=vec, vec_mom=vec_mom, vec_grad=vec_grad)


def _views(flat, offs, shapes, base=0):
    return [flat[base + o:base + o + m * n].view(m, n) for o, (m, n) in zip(offs, shapes)]


class _Lent:
    """A state tensor of a context, in place (Jorge.state_ptr), as the array interface torch reads."""

    def __init__(self, ctx, ptr, ld, rows, cols):
        self.owner = ctx
        self.__cuda_array_interface__ = {"shape": (rows, cols), "strides": (4 * ld, 4), "typestr": "<f4",
                                         "data": (ptr, False), "version": 2}


def _lent(ctx, layer, kind, rows, cols):
    ptr, ld = ctx.state_ptr(layer, kind)
    view = torch.as_tensor(_Lent(ctx, ptr, ld, rows, cols), device="cuda")
    view.owner = ctx           # the memory is the context's: it lives as long as the view
    return view


def _shown(num_layers):
    """Layers whose state a pass returns: all, or SHOWN of them evenly spread."""
    if num_layers <= SHOWN:
        return list(range(num_layers))
    return [round(i * (num_layers - 1) / (SHOWN - 1)) for i in range(SHOWN)]


def _restore(ctx, x):
    for l in range(len(x["shapes"])):
        ctx.set_state(l, "L", x["factors"][l][0])
        ctx.set_state(l, "R", x["factors"][l][1])
        ctx.set_state(l, "mom", x["moms"][l])
        ctx.set_state(l, "mom_sgd", x["msgds"][l])
    ctx.t = 100        # mid-run: the next step updates at interval 1, not at NO_UPDATE


def prepare(case, seed):
    x = _inputs(case, seed)
    shapes, entry = x["shapes"], case["entry"]
    interval = 1 if case["update"] else NO_UPDATE
    params = _views(x["theta"], x["offs"], shapes)
    cycle = _cycle(case)
    grads = [_views(x["noise"], x["offs"], shapes, _shift(i)) for i in range(cycle)]
    state = {"entry": entry, "at": 0, "params": params, "grads": grads, "keep": x["noise"]}
    if entry == "noalloc":
        (L, R), mom, msgd = x["factors"][0], x["moms"][0], x["msgds"][0]
        t = 1 if case["update"] else 2
        state.update(t=t, options=dict(precond_interval=interval), held=(L, R, mom, msgd),
                     out=[x["theta"], L, R, mom, msgd])
        return state
    if entry == "optimizer":
        vecs = [torch.nn.Parameter(x["vec"][o:o + n]) for o, n in zip(x["voffs"], vectors_of(case))]
        mats = [torch.nn.Parameter(p) for p in params]
        opt = JorgeOptimizer(mats + vecs, precond_interval=interval, **HYPER)
        for p, o in zip(vecs, x["voffs"]):
            opt.state[p]["momentum_buffer"] = x["vec_mom"][o:o + p.numel()].clone()
            p.grad = x["vec_grad"][o:o + p.numel()]
        for p, g in zip(mats, grads[0]):
            p.grad = g
        ctx = opt.ctx
        state.update(opt=opt, mats=mats, vecs=vecs)
    else:
        ctx = Jorge(shapes, precond_interval=interval)
        state["param_ptrs"] = Jorge.pointer_array(params)
        state["grad_ptrs"] = [Jorge.pointer_array(g) for g in grads]
    _restore(ctx, x)
    out = [x["theta"]] + ([x["vec"]] if entry == "optimizer" else [])
    for l in _shown(len(shapes)):
        m, n = shapes[l]
        out += [_lent(ctx, l, k, r, c) for k, r, c in (("L", m, m), ("R", n, n), ("mom", m, n), ("mom_sgd", m, n))]
    state.update(ctx=ctx, out=out)
    return state


def run(state):
    entry, i = state["entry"], state["at"]
    state["at"] = (i + 1) % len(state["grads"])
    if entry == "step":
        state["ctx"].step(state["params"], state["grads"][i], **HYPER)
    elif entry == "ptrs":
        state["ctx"].step_ptrs(state["param_ptrs"], state["grad_ptrs"][i], **HYPER)
    elif entry == "optimizer":
        if len(state["grads"]) > 1:
            for p, g in zip(state["mats"], state["grads"][i]):
                p.grad = g
        state["opt"].step()
    else:
        L, R, mom, msgd = state["held"]
        Jorge.step_noalloc(state["t"], state["params"][0], state["grads"][i][0], L, R, mom, msgd, **HYPER,
                           **state["options"])
    return state["out"]


# ------------------------------------------------------------------ the same in 64 bits

def _updated(A, M, beta2):
    """One factor update of Algorithm 2 with the clamped dynamic beta, symmetrized."""
    A2 = A @ A
    X = (A2 @ A2) @ M
    nu = float(torch.linalg.norm(X))
    c, s = ((1.0 / nu, (1.0 + 1.0 / nu) ** 0.25) if nu > beta2 / (1.0 - beta2)
            else ((1.0 - beta2) / beta2, beta2 ** -0.25))
    P = (-0.25 * c) * X + (0.15625 * c * c) * (X @ X)
    P.diagonal().add_(1.0)
    Z = s * (A @ P)
    return 0.5 * (Z + Z.t())


def exact(case, seed):
    x = _inputs(case, seed)
    lr, beta2, beta1, wd = HYPER["lr"], HYPER["beta2"], HYPER["beta1"], HYPER["weight_decay"]
    shapes = x["shapes"]
    theta = x["theta"].double()
    shown = set(_shown(len(shapes)))
    states = []
    for l, ((m, n), o) in enumerate(zip(shapes, x["offs"])):
        G = x["noise"][o:o + m * n].view(m, n).double()
        L, R = (f.double() for f in x["factors"][l])
        x["factors"][l] = None
        if case["update"]:
            L, R = _updated(L, G @ G.t(), beta2), _updated(R, G.t() @ G, beta2)
        mom = beta1 * x["moms"][l].double() + (1.0 - beta1) * ((L @ G) @ R)
        msgd = beta1 * x["msgds"][l].double() + G
        g = lr * float(torch.linalg.norm(msgd)) / float(torch.linalg.norm(mom))
        t = theta[o:o + m * n]
        t.copy_(t * (1.0 - lr * wd) - g * mom.reshape(-1))
        if l in shown:
            states += [L, R, mom, msgd]
    if case["entry"] != "optimizer":
        return [theta] + states
    vec = x["vec"].double()
    for o, n in zip(x["voffs"], vectors_of(case)):
        vec[o:o + n] -= lr * (beta1 * x["vec_mom"][o:o + n].double() + x["vec_grad"][o:o + n].double())
    return [theta, vec] + states


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: each gradient read, parameters, momenta and factors read and (factors: in an updating pass)
    written. Flops: each factor update in the cheapest of the three known orders of the same result (the
    paper's powers; through the gradient, low rank; that with A^2 formed), symmetric products once, and L G R."""
    nbytes = flops = 0.0
    for m, n in shapes_of(case):
        nbytes += 4.0 * (7 * m * n + (2 if case["update"] else 1) * (m * m + n * n))
        flops += 2.0 * m * n * (m + n)
        for d, k in ((float(m), float(n)), (float(n), float(m))) if case["update"] else ():
            flops += min(8 * d ** 3 + d * d * k, 12 * d * d * k + 5 * d * k * k, d ** 3 + 8 * d * d * k + 5 * d * k * k)
    return {"bytes": nbytes + 20.0 * sum(vectors_of(case)), "flops": flops}


def tolerance(case):
    """fp32 sums: against 64 bits the path is at most 8e-7 off on the 4096-wide layers and 3.5e-7 elsewhere (relative
    2-norm of any output); another order of the sums moves the outputs by as much."""
    return {"rel": 4e-6, "max": 2e-4}
