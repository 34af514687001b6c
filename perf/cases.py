"""The work that a user of this library has it do, as cases that can be timed.

Every case is one call sequence of a training step through the public entry points of
`paper_1806_04090_amd.binding`: a worker encodes its gradient and decodes it again ("svd", "entrywise", "lq"), a
parameter server combines the messages of its workers ("server"), or a caller with a decomposition of its own asks
for Algorithm 1 alone ("probabilities").  `listed()` names the sizes of the library's own configurations with the
smallest and the largest calls beside them; `draw(rng)` gives further sizes of the same ranges, odd ones among them.

Gradients are synthetic and made on the GPU from the seed alone: a few dominant singular values over a noise floor for
matrices, N(0, 1e-3^2) with one entry in a thousand a hundred times larger for flat gradients (the distributions of
`inputs.py`).  Messages, outputs and the context are what a training loop keeps from step to step.
"""
from __future__ import annotations

import math

import torch

from paper_1806_04090_amd import binding, inputs

_contexts = {}


def _context():
    """One context for the process, as a training loop has."""
    if "ctx" not in _contexts:
        _contexts["ctx"] = binding.Context(0)
    return _contexts["ctx"]


# ------------------------------------------------------------------------------------------------ layer sets

def _vgg11bn_matrices():
    """VGG-11-BN in the out x (in*k*k) reshape."""
    return [(x, y * k * k) for x, y, k in inputs.VGG11BN_CONVS] + list(inputs.VGG11BN_FCS)


_SETS = {
    "resnet18": lambda: list(inputs.RESNET18_SHAPES),
    "resnet18_section6": lambda: list(inputs.RESNET18_SECTION6_SHAPES),
    "vgg11bn_section6": lambda: list(inputs.VGG11BN_SECTION6_SHAPES),
    "vgg11bn": _vgg11bn_matrices,
}


def _shapes(layers: str):
    """A named layer set, or a list like "64x576,512x4608*64" (the number behind * is how often)."""
    if layers in _SETS:
        return _SETS[layers]()
    out = []
    for part in layers.split(","):
        size, _, times = part.partition("*")
        rows, cols = size.split("x")
        out += [(int(rows), int(cols))] * int(times or 1)
    return out


def _lengths(text: str):
    """Segment lengths: "64,512*4" is one of 64 and four of 512."""
    out = []
    for part in text.split(","):
        n, _, times = part.partition("*")
        out += [int(n)] * int(times or 1)
    return out


# ------------------------------------------------------------------------------------------------ the cases

def listed():
    n = inputs.RESNET18_PARAMETERS
    return [
        # one 3x3 convolution, 64 -> 64 channels: the smallest call that is a matrix, a latency
        {"name": "svd_64x576", "kind": "svd", "layers": "64x576", "s": 2.0, "signal": 4, "noise": 1e-2},
        # the gradient of ResNet-18, the library's headline step
        {"name": "svd_resnet18", "kind": "svd", "layers": "resnet18", "s": 3.0, "signal": 8, "noise": 1e-3},
        # 64 deep convolutions of a VGG-style network in one call: the largest one, every compute unit busy
        {"name": "svd_512x4608_x64", "kind": "svd", "layers": "512x4608*64", "s": 4.0, "signal": 16, "noise": 1e-2},
        # layers whose sizes fit no tile: wide and tall, a few rows over a block boundary
        {"name": "svd_ragged", "kind": "svd", "layers": "601x1237,1301x333,129x3001,47x799,10x1001", "s": 3.0,
         "signal": 8, "noise": 1e-3},
        # ResNet-18 in the paper's own reshape (Section 6): 18 columns, up to 131072 rows
        {"name": "svd_resnet18_section6", "kind": "svd", "layers": "resnet18_section6", "s": 3.0, "signal": 8,
         "noise": 1e-3},
        # the parameter server's average of 16 workers' ResNet-18 messages
        {"name": "server_average_16", "kind": "server", "layers": "resnet18", "workers": 16, "s": 3.0, "update": False},
        # the parameter server's step on VGG-11-BN, 8 workers: the average is applied to the parameters in place
        {"name": "server_update_8", "kind": "server", "layers": "vgg11bn", "workers": 8, "s": 3.0, "update": True},
        # the batch-norm and bias scalars of ResNet-18: a flat gradient so short that launches are all that counts
        {"name": "entrywise_9610", "kind": "entrywise", "n": n - inputs.RESNET18_ELEMENTS, "keep": 0.01},
        # the flat gradient of ResNet-18
        {"name": "entrywise_resnet18", "kind": "entrywise", "n": n, "keep": 0.01},
        # a gradient of a quarter of a billion elements, of odd length
        {"name": "entrywise_268M", "kind": "entrywise", "n": (1 << 28) + 3, "keep": 0.01},
        # 1-bit QSGD of the flat gradient of ResNet-18 (Section 4, q = 2)
        {"name": "lq2_resnet18", "kind": "lq", "n": n, "q": 2.0},
        # Algorithm 1 alone: the singular values of the ResNet-18 layers and one long vector of coefficients
        {"name": "probabilities_mixed", "kind": "probabilities",
         "lengths": "27,64*5,128*4,256*6,512*4,10,1000003", "s": 3.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _matrix(rng, short_lo, short_hi, long_hi):
    short = _log_int(rng, short_lo, short_hi)
    long = _log_int(rng, short, max(short + 1, long_hi))
    return (short, long) if rng.random() < 0.7 else (long, short)


def draw(rng):
    kind = rng.choice(["svd", "svd", "thin", "server", "entrywise", "entrywise", "lq", "probabilities"])
    if kind == "svd":
        # layer sets from one small matrix to some dozens, up to about the elements of ResNet-18 times four
        count = _log_int(rng, 1, 40)
        parts, budget = [], 40_000_000
        for _ in range(count):
            m, k = _matrix(rng, 33, 640, 4608)
            if m * k > budget:
                break
            budget -= m * k
            parts.append("%dx%d" % (m, k))
        return {"kind": "svd", "layers": ",".join(parts), "s": round(rng.uniform(1.0, 6.0), 2), "signal": rng.randint(2, 16),
                "noise": round(10.0 ** rng.uniform(-3.0, -2.0), 5)}
    if kind == "thin":
        # matrices of at most 32 columns (the Section 6 reshape has 18 and 2)
        parts = []
        for _ in range(_log_int(rng, 1, 24)):
            cols = rng.choice([2, 18, 18, 18, rng.randint(3, 32)])
            parts.append("%dx%d" % (_log_int(rng, 64, 131072), cols))
        return {"kind": "svd", "layers": ",".join(parts), "s": round(rng.uniform(1.0, 4.0), 2), "signal": rng.randint(2, 8),
                "noise": round(10.0 ** rng.uniform(-3.0, -2.0), 5)}
    if kind == "server":
        parts, budget = [], 12_000_000
        for _ in range(_log_int(rng, 1, 24)):
            m, k = _matrix(rng, 10, 640, 4608)
            if m * k > budget:
                break
            budget -= m * k
            parts.append("%dx%d" % (m, k))
        return {"kind": "server", "layers": ",".join(parts), "workers": _log_int(rng, 1, 16),
                "s": round(rng.uniform(1.0, 4.0), 2), "update": rng.random() < 0.5}
    if kind == "entrywise":
        return {"kind": "entrywise", "n": _log_int(rng, 1000, 1 << 28), "keep": round(10.0 ** rng.uniform(-3.0, -1.0), 5)}
    if kind == "lq":
        return {"kind": "lq", "n": _log_int(rng, 1000, 1 << 27), "q": rng.choice([2.0, "inf", 1.5])}
    parts = ["%d" % _log_int(rng, 2, 2048) for _ in range(_log_int(rng, 1, 60))]
    if rng.random() < 0.5:
        parts.append("%d" % _log_int(rng, 2049, 20_000_000))
    return {"kind": "probabilities", "lengths": ",".join(parts), "s": round(rng.uniform(1.0, 6.0), 2)}


# ------------------------------------------------------------------------------------------------ inputs

def _gradient_matrix(gen, m, k, signal, noise):
    """rank-`signal` geometric signal 0.5^j over N(0, noise^2)."""
    rank = min(signal, m, k)
    u = torch.randn(m, rank, generator=gen, device="cuda")
    v = torch.randn(rank, k, generator=gen, device="cuda")
    u /= u.norm(dim=0, keepdim=True)
    v /= v.norm(dim=1, keepdim=True)
    u *= 0.5 ** torch.arange(rank, device="cuda", dtype=torch.float32)
    g = torch.randn(m, k, generator=gen, device="cuda")
    g *= noise
    g += u @ v
    return g


def _flat_gradient(gen, n):
    """N(0, 1e-3^2), one entry in a thousand (at random places) a hundred times larger."""
    g = torch.randn(n, generator=gen, device="cuda")
    g *= 1e-3
    heavy = n // 1000
    if heavy:
        at = torch.randint(0, n, (heavy,), generator=gen, device="cuda")
        g[at] = 100.0 * g[at]
    return g


def _messages(shapes, s):
    """Message buffers for a layer set; the counts, indices and weights of all layers lie side by side."""
    caps = [binding.default_capacity(s, min(m, k)) for m, k in shapes]
    count = torch.zeros(len(shapes), dtype=torch.int32, device="cuda")
    idx = torch.zeros(sum(caps), dtype=torch.int32, device="cuda")
    w = torch.zeros(sum(caps), dtype=torch.float32, device="cuda")
    msgs, at = [], 0
    for j, ((m, k), cap) in enumerate(zip(shapes, caps)):
        msgs.append(binding.SvdMessage(m, k, cap, count[j:j + 1], idx[at:at + cap], w[at:at + cap],
                                       torch.zeros(cap, m, device="cuda"), torch.zeros(cap, k, device="cuda")))
        at += cap
    return msgs, count, idx, w


def _dense(shapes):
    """One flat buffer for a layer set and the matrices in it."""
    flat = torch.zeros(sum(m * k for m, k in shapes), device="cuda")
    views, at = [], 0
    for m, k in shapes:
        views.append(flat[at:at + m * k].view(m, k))
        at += m * k
    return flat, views


def prepare(case, seed):
    ctx = _context()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    state = {"case": case, "ctx": ctx, "kind": kind, "seed": int(seed)}
    if kind == "svd":
        shapes = _shapes(case["layers"])
        state["mats"] = [_gradient_matrix(gen, m, k, case["signal"], case["noise"]) for m, k in shapes]
        state["msgs"], state["count"], state["idx"], state["w"] = _messages(shapes, case["s"])
        state["flat"], state["outs"] = _dense(shapes)
        state["groups"] = [[m] for m in state["msgs"]]
    elif kind == "server":
        # the workers' messages, as they arrive at the server
        shapes, workers = _shapes(case["layers"]), case["workers"]
        per_worker = []
        for p in range(workers):
            mats = [_gradient_matrix(gen, m, k, 8, 1e-3) for m, k in shapes]
            msgs = _messages(shapes, case["s"])[0]
            binding.atomo_encode_svd(ctx, mats, case["s"], int(seed), inputs.worker_stream(p, 0), msgs=msgs)
            per_worker.append(msgs)
        state["groups"] = [[per_worker[p][j] for p in range(workers)] for j in range(len(shapes))]
        state["flat"], state["outs"] = _dense(shapes)
        if case["update"]:
            state["flat"].normal_(0.0, 0.05, generator=gen)      # the parameters
    elif kind == "entrywise":
        n = case["n"]
        state["g"] = _flat_gradient(gen, n)
        state["s"] = case["keep"] * n
        state["msg"] = binding.alloc_entrywise_message(n, binding.default_capacity(state["s"], n), "cuda")
        state["out"] = torch.zeros(n, device="cuda")
    elif kind == "lq":
        n = case["n"]
        state["q"] = float(case["q"])
        state["g"] = _flat_gradient(gen, n)
        state["msg"] = binding.alloc_lq_message(n, binding.lq_capacity(n, state["q"]), "cuda")
        state["out"] = torch.zeros(n, device="cuda")
    else:
        lengths = _lengths(case["lengths"])
        offsets = [0]
        for n in lengths:
            offsets.append(offsets[-1] + n)
        lam = torch.randn(offsets[-1], generator=gen, device="cuda").abs_()
        lam *= torch.rand(offsets[-1], generator=gen, device="cuda").pow_(4.0)      # a few large ones over many small
        state["lam"], state["offsets"], state["p"] = lam, offsets, torch.zeros_like(lam)
    return state


# ------------------------------------------------------------------------------------------------ one pass

def run(state):
    ctx, case, kind = state["ctx"], state["case"], state["kind"]
    if kind == "svd":
        binding.atomo_encode_svd(ctx, state["mats"], case["s"], state["seed"], 0, msgs=state["msgs"], adaptive=1)
        binding.atomo_decode_svd_batch(ctx, state["groups"], 1.0, outs=state["outs"])
        return {"count": state["count"], "idx": state["idx"], "w": state["w"], "dense": state["flat"]}
    if kind == "server":
        if case["update"]:
            binding.atomo_apply_svd_batch(ctx, state["groups"], -0.01 / case["workers"], state["outs"])
        else:
            binding.atomo_decode_svd_batch(ctx, state["groups"], 1.0 / case["workers"], outs=state["outs"])
        return state["flat"]
    if kind == "entrywise":
        msg = binding.atomo_encode_entrywise(ctx, state["g"], state["s"], state["seed"], 0, msg=state["msg"])
        out = binding.atomo_decode(ctx, [msg], out=state["out"])
        return {"count": msg.count, "idx": msg.idx, "val": msg.val, "dense": out}
    if kind == "lq":
        msg = binding.atomo_encode_lq(ctx, state["g"], state["q"], state["seed"], 0, msg=state["msg"])
        out = binding.atomo_decode(ctx, [msg], out=state["out"])
        return {"count": msg.count, "idx": msg.idx, "norm": msg.norm, "dense": out}
    return binding.atomo_probabilities(ctx, state["lam"], state["offsets"], case["s"], out=state["p"])


# ------------------------------------------------------------------------------------------------ what a pass needs

def work(case):
    kind = case["kind"]
    if kind == "svd":
        # each gradient read once, each dense output written once, about s atoms written and read; the flops are those
        # of a reduction to bidiagonal form of the r x M matrix through its Gram matrix (M r^2 for one triangle of it,
        # 4/3 r^3 to reduce it) and of the kept atoms (formed and decoded)
        nbytes = flops = 0.0
        for m, k in _shapes(case["layers"]):
            r, long = min(m, k), max(m, k)
            atoms = min(case["s"], r)
            nbytes += 8.0 * m * k + 8.0 * atoms * (m + k + 2)
            flops += long * r * (r + 1.0) + 4.0 / 3.0 * r ** 3 + 4.0 * atoms * m * k
        return {"bytes": nbytes, "flops": flops}
    if kind == "server":
        nbytes = flops = 0.0
        for m, k in _shapes(case["layers"]):
            atoms = case["workers"] * min(case["s"], m, k)
            nbytes += (8.0 if case["update"] else 4.0) * m * k + 4.0 * atoms * (m + k + 1)
            flops += 2.0 * atoms * m * k
        return {"bytes": nbytes, "flops": flops}
    if kind == "entrywise":
        # the water level needs all of g before the first draw, but g can be kept on chip or read again: counted once
        n, kept = case["n"], case["n"] * case["keep"]
        return {"bytes": 8.0 * n + 16.0 * kept, "flops": 2.0 * n}
    if kind == "lq":
        n, q = case["n"], float(case["q"])
        # kept = |g|_1 / |g|_q of this distribution
        def power_sum(x):
            normal = 2.0 ** (x / 2.0) * math.gamma((x + 1.0) / 2.0) / math.sqrt(math.pi)
            return n * normal * (1e-3 ** x + 1e-3 * 0.1 ** x)

        norm = 0.4 if math.isinf(q) else power_sum(q) ** (1.0 / q)
        return {"bytes": 8.0 * n + 8.0 * min(n, power_sum(1.0) / norm), "flops": 2.0 * n}
    total = sum(_lengths(case["lengths"]))
    return {"bytes": 8.0 * total, "flops": 2.0 * total}


def tolerance(case):
    if case["kind"] in ("svd", "server"):
        # Counts and indices are the same, weights agree to 1e-6.  A decoded gradient is made of a few singular vectors
        # that were drawn from the noise floor, where neighbouring singular values differ by about 1e-4 of the largest:
        # inside such a cluster two fp32 decompositions, each with singular-pair residuals of 1e-6, give vectors that
        # differ by 1e-3 to 5e-3 (single entries by up to 0.2 of the root mean square; other block orders and stopping
        # rules of the same Jacobi iteration, in fp32).
        return {"rel": 1e-2, "max": 0.4}
    # sums are exact or in double precision, every value is rounded to fp32 once
    return {"rel": 1e-6}
