"""The work that a user of this library has it do, as measurable cases.

A case is one outer step (``IsoLoCoPlan.aggregate`` or ``aggregate_static``)
over a parameter layout: either one matrix and a vector, or a LLaMA-style model
(per block q, k, v, o of d x d, gate and up of f x d, down of d x f and two
gains, and one tied V x d embedding).  Inputs follow the synthetic workloads
of the benchmark: theta ~ N(0, 0.02^2), worker k's pseudo-gradient a shared
low-rank component plus its own Gaussian noise, replicas rounded to float32 or
bfloat16; the momentum is the one of a running training (not zero).

A pass restores theta and the momentum (one copy) and runs the step: a step on
its own result would meet a pseudo-gradient that the last step has made
isotropic, which no training shows.
"""
import math

import torch

import paper_2607_03011_amd as iso

ISO, AVG = iso.ISOLOCO_KIND_ISO, iso.ISOLOCO_KIND_AVG

ALPHA, OUTER_LR, MU = 1.0, 0.7, 0.9
THETA_STD, NOISE_STD, MOMENTUM_STD, SHARED = 0.02, 1e-4, 3e-4, 1e-3

# plan options of the variants: the paper's step (the library's defaults), its
# fast variant (five Newton-Schulz steps, RMS scale) and its clip_high
VARIANTS = {
    "exact": {},
    "fast": {"orth": iso.ISOLOCO_ORTH_NS5, "scale": iso.ISOLOCO_SCALE_RMS},
    "clip_high": {"clip": iso.ISOLOCO_CLIP_HIGH},
}


def _model(name, blocks, d, f, vocab, K, dtype, variant="exact", entry="aggregate", embedding="iso"):
    return {"name": name, "kind": "model", "blocks": blocks, "d": d, "f": f, "vocab": vocab, "K": K,
            "dtype": dtype, "variant": variant, "entry": entry, "embedding": embedding}


def _single(name, rows, cols, vector, K, dtype, variant="exact", entry="aggregate"):
    return {"name": name, "kind": "single", "rows": rows, "cols": cols, "vector": vector, "K": K,
            "dtype": dtype, "variant": variant, "entry": entry}


def listed():
    return [
        # the smallest call: one adapter-sized matrix, where launches and latency count
        _single("single-128x64-K4", 128, 64, 64, 4, "f32"),
        # one decoder block, as a shard of a model or a first experiment
        _model("block-d768-K8", 1, 768, 2048, 0, 8, "f32"),
        # the entry point for callers that cannot allocate, bf16 replicas
        _model("block-d512-K4-bf16-static", 1, 512, 1408, 0, 4, "bf16", entry="static"),
        # odd and ragged sizes: no dimension of the MLP is a multiple of anything
        _model("ragged-4L-d612-f1637-K6", 4, 612, 1637, 0, 6, "f32"),
        # the clip_high variant, two blocks
        _model("2L-d768-K8-clip_high", 2, 768, 2048, 0, 8, "f32", variant="clip_high"),
        # one large square matrix
        _single("single-4096x4096-K8-bf16", 4096, 4096, 4096, 8, "bf16"),
        # the benchmark: 109.5M parameters, float32 replicas
        _model("12L-d768-V32000-K16", 12, 768, 2048, 32000, 16, "f32"),
        # the paper's fast variant on the same model
        _model("12L-d768-V32000-K16-fast", 12, 768, 2048, 32000, 16, "f32", variant="fast"),
        # 341M parameters, bf16 replicas of 32 workers
        _model("24L-d1024-V32000-K32-bf16", 24, 1024, 2816, 32000, 32, "bf16"),
        # wide blocks (d = 2048): the largest products
        _model("8L-d2048-V32000-K16-bf16", 8, 2048, 5632, 32000, 16, "bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: widths from 16 to 2048 (4096 for one matrix), one in
    three of them odd, the others multiples of 64 where they are wide; up to
    16 blocks, with or without an embedding; 2 to 64 workers."""
    def size(lo, hi):
        v = _log(rng, lo, hi)
        return v if rng.random() < 1 / 3 else max(16, v // 64 * 64 if v >= 192 else v // 16 * 16)

    top = [work(c) for c in listed()]
    most = {k: max(w[k] for w in top) for k in ("bytes", "flops")}
    while True:
        K, dtype = _log(rng, 2, 64), rng.choice(["f32", "bf16"])
        variant = rng.choice(["exact"] * 6 + ["fast", "clip_high"])
        if rng.random() < 0.25:
            c = _single("", size(16, 4096), size(16, 4096), _log(rng, 16, 4096), K, dtype, variant)
        else:
            d = size(64, 2048)
            c = _model("", _log(rng, 1, 16), d, int(d * rng.uniform(2, 4)) if rng.random() < 1 / 3 else
                       max(64, int(d * 8 / 3) // 64 * 64), rng.choice([0, 0, _log(rng, 1000, 32000)]), K, dtype,
                       variant, embedding=rng.choice(["iso", "iso", "iso", "avg"]))
            if c["blocks"] == 1 and not c["vocab"] and d <= 512 and variant == "exact" and rng.random() < 0.5:
                c["entry"] = "static"
        del c["name"]
        w = work(c)
        if all(w[k] <= most[k] for k in most):
            return c


def _layout(case):
    if case["kind"] == "single":
        shapes = [(case["rows"], case["cols"], ISO), (case["vector"], 1, AVG)]
    else:
        d, f = case["d"], case["f"]
        shapes = []
        for _ in range(case["blocks"]):
            shapes += [(d, 1, AVG)] + [(d, d, ISO)] * 4 + [(d, 1, AVG)] + [(f, d, ISO)] * 2 + [(d, f, ISO)]
        if case["vocab"]:
            shapes.append((case["vocab"], d, ISO if case["embedding"] == "iso" else AVG))
    layout, off = [], 0
    for rows, cols, kind in shapes:
        layout.append((off, rows, cols, kind))
        off += rows * cols
    return layout, off


def _inputs(case, seed):
    """theta, momentum and the [K, n] replicas (rows 256-byte aligned)."""
    layout, n = _layout(case)
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    K = case["K"]
    start = torch.randn((2, (n + 127) // 128 * 128), generator=g, device=dev)
    start[0].mul_(THETA_STD)
    start[1].mul_(MOMENTUM_STD)
    theta = start[0, :n]
    workers = torch.empty((K, (n + 127) // 128 * 128), device=dev,
                          dtype=torch.float32 if case["dtype"] == "f32" else torch.bfloat16)[:, :n]
    for off, rows, cols, kind in layout:
        if kind == ISO:
            r = min(64, rows, cols)
            shared = torch.randn(rows, r, generator=g, device=dev) @ torch.randn(r, cols, generator=g, device=dev)
            shared = shared.mul_(SHARED / math.sqrt(r)).reshape(-1)
        else:
            shared = torch.randn(rows * cols, generator=g, device=dev).mul_(SHARED)
        base = theta[off:off + rows * cols] - shared
        for k in range(K):
            noise = torch.randn(rows * cols, generator=g, device=dev)
            workers[k, off:off + rows * cols] = torch.add(base, noise, alpha=-NOISE_STD)
    return layout, n, start, workers


def prepare(case, seed):
    layout, n, start, workers = _inputs(case, seed)
    static = case["entry"] == "static"
    plan = iso.IsoLoCoPlan(layout, n, case["K"], iso.ISOLOCO_F32 if case["dtype"] == "f32" else iso.ISOLOCO_BF16,
                           opts=VARIANTS[case["variant"]] or None, workspace=not static)
    current = torch.empty_like(start)
    return {"plan": plan, "step": plan.aggregate_static if static else plan.aggregate, "start": start,
            "current": current, "theta": current[0, :n], "momentum": current[1, :n],
            "workers": [workers[k] for k in range(case["K"])]}


def run(state):
    state["current"].copy_(state["start"])
    state["step"](state["theta"], state["workers"], state["momentum"], ALPHA, OUTER_LR, MU)
    return {"theta": state["theta"], "momentum": state["momentum"]}


def work(case):
    """Bytes: the replicas, theta and the momentum read once, theta and the
    momentum written once.  Flops: the polar iteration's products, in float32
    flops: per step of an m x n matrix (m >= n) the symmetric Gram n (n + 1) m,
    the symmetric square n (n + 1) n and the product 2 m n^2, over the 7 steps
    that a tall matrix (m >= 2 n) of these spectra needs, or the 13 of a square
    one (5 in the fast variant, two iterations in clip_high)."""
    layout, n = _layout(case)
    flops = 0
    for _, rows, cols, kind in layout:
        if kind == ISO:
            m, k = max(rows, cols), min(rows, cols)
            steps = 5 if case["variant"] == "fast" else 7 if m >= 2 * k else 13
            flops += steps * (k * (k + 1) * m + k * (k + 1) * k + 2 * m * k * k) * (2 if case["variant"] == "clip_high"
                                                                                   else 1)
    return {"bytes": n * (case["K"] * (4 if case["dtype"] == "f32" else 2) + 16), "flops": flops}


def tolerance(case):
    """The products take float32 operands as two or three bfloat16 parts, with
    float32 sums (relative error 2^-16 per product); square noise-like matrices
    amplify it through their small singular values: against float64 the listed
    cases are 1e-5 to 4e-5 off in the momentum, and a matrix with an unusually
    small singular value several times that."""
    return {"rel": 4e-4, "max": 2e-2}


def _polar(x):
    """The orthogonal polar factor of a float64 matrix by the cubic Newton-Schulz iteration."""
    tall = x if x.shape[0] >= x.shape[1] else x.T.contiguous()
    q = tall / torch.linalg.norm(tall)
    q = q / torch.linalg.norm(q.T @ q).sqrt()
    eye = torch.eye(q.shape[1], dtype=q.dtype, device=q.device)
    for k in range(120):
        a = q.T @ q
        if k % 8 == 7 and torch.linalg.norm(a - eye).item() < 1e-11 * math.sqrt(q.shape[1]):
            break
        q = torch.addmm(q, q, a, beta=1.5, alpha=-0.5)
    return q if x.shape[0] >= x.shape[1] else q.T


def _correct(delta, variant):
    r = min(delta.shape)
    if variant == "fast":
        x = delta / torch.linalg.norm(delta)
        x = x if x.shape[0] >= x.shape[1] else x.T
        for _ in range(5):
            a = x.T @ x
            x = 3.4445 * x - 4.7750 * (x @ a) + 2.0315 * (x @ (a @ a))
        x = x if delta.shape[0] >= delta.shape[1] else x.T
        return torch.linalg.norm(delta) / math.sqrt(r) * x
    q = _polar(delta)
    mean = (q * delta).sum() / r
    if variant == "exact":
        return mean * q
    # clip_high: the singular values above the mean set to the mean.  With
    # E = Delta - mean Q and its polar factor Q2, |E| = Q Q2^T E holds
    # |sigma - mean|, and min(sigma, mean) = mean + ((sigma - mean) - |sigma - mean|) / 2
    e = delta - mean * q
    q2 = _polar(e)
    return mean * q + (e - (q @ (q2.T @ e) if q.shape[0] >= q.shape[1] else (e @ q2.T) @ q)) / 2


def exact(case, seed):
    layout, n, start, workers = _inputs(case, seed)
    theta, mom = start[0, :n].double(), start[1, :n].double()
    for off, rows, cols, kind in layout:
        span = slice(off, off + rows * cols)
        d = torch.zeros(rows * cols, dtype=torch.float64, device=theta.device)
        for k in range(case["K"]):
            d += theta[span] - workers[k, span].double()
        d /= case["K"]
        if kind == ISO:
            d = _correct(d.reshape(rows, cols), case["variant"]).reshape(-1) * ALPHA
        mom[span] = MU * mom[span] + d
        theta[span] -= OUTER_LR * (d + MU * mom[span])
    return {"theta": theta, "momentum": mom}
