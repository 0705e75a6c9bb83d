"""The work that a user of this library has it do, as measurable cases.

A case is one pass through the public entry points of
`paper_2310_07177_amd` (the logits path of online speculative decoding):
verification of a batch of proposals, the distillation loss and gradient, one
speculative step that does both, tree verification and token sampling.

A case with "graph" set is one that a serving program captures once into a
HIP graph and replays for every step (the decode loop: its calls are short, so
launches would bound it); prepare() captures it, as the program would at
start-up.  The others call the entry points eagerly, as a script or a training
loop does.

Logits follow the recipe of the synthetic workloads in
`paper_2310_07177_amd/synth.py` (target ~ N(0, std^2), draft = scale * target
+ N(0, noise^2), proposals drawn from the draft), made on the GPU with torch's
seeded generator.
"""
import math

import torch

import paper_2310_07177_amd as osd
from paper_2310_07177_amd import synth

DEV = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
# The largest row of the whole-row entry points and of the tree call.
MAX_V = {"bf16": 131072, "f32": 65536}
MAX_TREE_V = {"bf16": 32768, "f32": 16384}


# --------------------------------------------------------------------------
# The cases
# --------------------------------------------------------------------------

def listed():
    return [
        # One user's stream, four proposals, called from Python: the smallest
        # call, where latency and host time count.
        dict(name="verify_single", op="verify", B=1, K=4, V=32000, dtype="bf16", T=1.0, std=3.0, scale=1.0,
             noise=1.0, ragged=False, graph=False),
        # A whole speculative step of a small serving batch: five proposal
        # draws, then verification with the distillation of the rejected rows.
        dict(name="spec_step_small", op="spec", B=8, K=5, V=32000, dtype="bf16", T=1.0, std=3.0, scale=1.0,
             noise=1.0, ragged=False, kind="fkl", beta=0.5, graph=True),
        # Verification in the decode loop of a full batch.
        dict(name="verify_batch", op="verify", B=64, K=8, V=32128, dtype="bf16", T=0.7, std=2.5, scale=0.7,
             noise=1.5, ragged=False, graph=True),
        # The same batch decoded greedily.
        dict(name="verify_greedy", op="verify", B=64, K=8, V=32128, dtype="bf16", T=0.0, std=2.5, scale=0.7,
             noise=1.5, ragged=False, graph=True),
        # A vocabulary with a few added tokens (rows no longer 16-byte
        # aligned), proposals of ragged lengths.
        dict(name="verify_added_tokens", op="verify", B=32, K=8, V=32003, dtype="bf16", T=1.0, std=3.0, scale=1.0,
             noise=1.0, ragged=True, graph=False),
        # The online update of a large-vocabulary model: verification, then
        # the loss and gradient at each first rejection.
        dict(name="step_large_vocab", op="rejected", B=256, K=8, V=128256, dtype="bf16", T=0.8, std=3.0, scale=1.0,
             noise=1.0, ragged=True, kind="fkl", beta=0.5, graph=False),
        # Verification and distillation of every position in one call.
        dict(name="step_all_rows", op="step", B=64, K=8, V=32128, dtype="bf16", T=0.7, std=2.5, scale=0.7,
             noise=1.5, ragged=False, kind="jsd", beta=0.5, graph=True),
        # The same for an odd vocabulary.
        dict(name="step_odd_vocab", op="step", B=32, K=6, V=50257, dtype="bf16", T=1.0, std=3.0, scale=1.0,
             noise=1.0, ragged=False, kind="rkl", beta=0.5, graph=False),
        # A training pass over the buffer of stored positions, 40 % of them
        # selected.
        dict(name="distill_buffer", op="distill", B=16384, K=1, V=32000, dtype="bf16", T=1.0, std=3.0, scale=1.0,
             noise=1.0, masked=0.4, kind="jsd", beta=0.5, graph=False),
        # Loss and gradient of float32 logits, every position.
        dict(name="distill_f32", op="distill", B=32, K=8, V=32000, dtype="f32", T=1.0, std=3.0, scale=1.0,
             noise=1.0, masked=1.0, kind="rkl", beta=0.5, graph=False),
        # Multi-candidate trees (branching 4, 3, 2, 1) of 64 nodes.
        dict(name="tree_batch", op="tree", B=16, N=64, V=32000, dtype="bf16", T=1.0, std=3.0, scale=1.0, noise=1.0,
             graph=True),
        # Tokens of the mixture of teacher and student, the source of
        # distillation data.
        dict(name="sample_mixed", op="sample", N=4096, V=32000, dtype="bf16", T=1.0, std=3.0, scale=1.0, noise=1.0,
             beta=0.5, graph=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# A drawn case moves at most this many bytes (below the largest listed case).
_DRAW_BYTES = 1.2e9


def draw(rng):
    while True:
        op = rng.choice(["verify", "verify", "spec", "rejected", "step", "step", "distill", "distill", "tree", "sample"])
        dtype = "f32" if rng.random() < 0.3 else "bf16"
        most = MAX_TREE_V[dtype] if op == "tree" else MAX_V[dtype]
        V = _log_uniform(rng, 16000 if most > 16384 else 8000, most)
        if rng.random() < 0.6:  # vocabularies are mostly padded
            V = V // 64 * 64
        case = dict(op=op, V=V, dtype=dtype, T=rng.choice([0.7, 0.8, 1.0]), std=rng.choice([2.0, 2.5, 3.0]),
                    scale=1.0, noise=rng.choice([0.25, 1.0, 2.0]))
        kind = rng.choice(["fkl", "rkl", "jsd"])
        beta = rng.choice([0.3, 0.5, 0.7])
        if op == "tree":
            case.update(B=_log_uniform(rng, 1, 32), N=_log_uniform(rng, 4, 64), graph=rng.random() < 0.5)
        elif op == "sample":
            mixed = rng.random() < 0.5
            case.update(N=_log_uniform(rng, 1, 8192 if mixed else 256), beta=beta if mixed else 0.0,
                        graph=not mixed and rng.random() < 0.5)
        elif op == "distill":
            case.update(B=_log_uniform(rng, 8, 8192), K=rng.choice([1, 4, 8]), kind=kind, beta=beta,
                        masked=rng.choice([0.4, 1.0]), graph=False)
        else:
            case.update(B=_log_uniform(rng, 1, 256), K=rng.randint(1, 8), ragged=op != "spec" and rng.random() < 0.4,
                        graph=rng.random() < 0.5)
            if op == "verify" and rng.random() < 0.25:
                case["T"] = 0.0
            if op != "verify":
                case.update(kind=kind, beta=beta)
            if op == "spec":
                case["graph"] = True
        if work(case)["bytes"] <= _DRAW_BYTES:
            return case


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _logits(case, g, lead, draft_lead=None):
    """Target rows, and draft rows for the first draft_lead[1] positions."""
    dt = DTYPES[case["dtype"]]
    t = torch.randn(*lead, case["V"], generator=g, device=DEV).mul_(case["std"])
    rows = t if draft_lead is None else t[:, :draft_lead[1]]
    d = (case["scale"] * rows).add_(torch.randn(rows.shape, generator=g, device=DEV), alpha=case["noise"])
    return t.to(dt), d.to(dt).contiguous()


def _proposals(rows, T, g):
    """One token ~ softmax(rows / T) per row (the argmax at T == 0)."""
    flat = rows.reshape(-1, rows.shape[-1])
    out = torch.empty(flat.shape[0], dtype=torch.int32, device=DEV)
    step = max(1, (64 << 20) // flat.shape[1])
    for r in range(0, flat.shape[0], step):
        x = flat[r:r + step].float()
        if T > 0:
            x = x / T - torch.empty_like(x).exponential_(generator=g).log_()
        out[r:r + step] = x.argmax(-1).to(torch.int32)
    return out.reshape(rows.shape[:-1])


def _inputs(case, seed):
    g = _generator(seed)
    op, V, T = case["op"], case["V"], case["T"]
    s = {"case": case}
    if op == "sample":
        N = case["N"]
        s["p"], s["q"] = _logits(case, g, (N,))
        if case["beta"] == 0.0:
            s["p"] = None
        s["u"] = torch.rand(N, generator=g, device=DEV)
        return s
    if op == "distill":
        B, K = case["B"], case["K"]
        s["t"], s["d"] = _logits(case, g, (B, K))
        s["mask"] = None
        if case["masked"] < 1.0:
            s["mask"] = (torch.rand(B, K, generator=g, device=DEV) < case["masked"]).to(torch.uint8)
        return s
    if op == "tree":
        B, N = case["B"], case["N"]
        s["t"], s["d"] = _logits(case, g, (B, N))
        parent = torch.from_numpy(synth.tree_parents((4, 3, 2, 1), N)).to(DEV)
        if parent.numel() < N:  # a tree of N nodes however large N is
            raise ValueError("the tree has fewer nodes than N")
        s["parent"] = parent.repeat(B, 1).contiguous()
        up = parent.clamp_min(0).long()
        s["tokens"] = torch.stack([_proposals(s["d"][b, up], T, g) for b in range(B)])
        s["ua"] = torch.rand(B, N, generator=g, device=DEV)
        s["ur"] = torch.rand(B, generator=g, device=DEV)
        return s
    B, K = case["B"], case["K"]
    s["t"], s["d"] = _logits(case, g, (B, K + 1), (B, K))
    s["tokens"] = None if op == "spec" else _proposals(s["d"], T, g)
    s["ua"] = torch.rand(B, K, generator=g, device=DEV)
    s["ur"] = torch.rand(B, generator=g, device=DEV)
    s["up"] = torch.rand(K, B, generator=g, device=DEV)
    s["len"] = torch.randint(1, K + 1, (B,), generator=g, device=DEV, dtype=torch.int32) if case["ragged"] else None
    return s


def _call(s):
    case = s["case"]
    op, T = case["op"], case["T"]
    if op == "verify":
        greedy = T == 0.0
        return osd.osd_verify(s["t"], None if greedy else s["d"], s["tokens"], None if greedy else s["ua"],
                              None if greedy else s["ur"], T, draft_len=s["len"])
    if op == "spec":
        B, K = case["B"], case["K"]
        drawn = torch.empty(K, B, dtype=torch.int32, device=DEV)
        for i in range(K):
            osd.osd_sample(None, s["d"][:, i, :], T, 0.0, s["up"][i], out=drawn[i])
        tokens = drawn.t().contiguous()
        return (tokens,) + tuple(osd.osd_verify_distill_rejected(s["t"], s["d"], tokens, s["ua"], s["ur"], T,
                                                                 case["kind"], case["beta"]))
    if op == "rejected":
        return osd.osd_verify_distill_rejected(s["t"], s["d"], s["tokens"], s["ua"], s["ur"], T, case["kind"],
                                               case["beta"], draft_len=s["len"])
    if op == "step":
        return osd.osd_verify_distill(s["t"], s["d"], s["tokens"], s["ua"], s["ur"], T, case["kind"], case["beta"],
                                      draft_len=s["len"])
    if op == "distill":
        return osd.osd_distill_loss_grad(s["t"], s["d"], case["kind"], case["beta"], T, mask=s["mask"])
    if op == "tree":
        return osd.osd_verify_tree(s["t"], s["d"], s["parent"], s["tokens"], s["ua"], s["ur"], T)
    return osd.osd_sample(s["p"], s["q"], T, case["beta"], s["u"])


_capture_stream = None


def prepare(case, seed):
    global _capture_stream
    s = _inputs(case, seed)
    if case["graph"]:
        if _capture_stream is None:
            _capture_stream = torch.cuda.Stream()
        _capture_stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(_capture_stream):  # one eager call: the workspace exists before the capture
            _call(s)
        torch.cuda.current_stream().wait_stream(_capture_stream)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"], stream=_capture_stream):
            s["out"] = _call(s)
    return s


def run(s):
    if "graph" in s:
        s["graph"].replay()
        return s["out"]
    return _call(s)


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    """Rows that the method needs, each read once, and the outputs.  (Ragged
    lengths count with their mean (K + 1) / 2, a verification reads the rows
    of every proposal and one bonus row per sequence.)"""
    op, V = case["op"], case["V"]
    row = V * (2 if case["dtype"] == "bf16" else 4)
    if op == "sample":
        two = 0.0 < case["beta"] < 1.0
        rows = case["N"] * (2 if two else 1)
        return dict(bytes=rows * row + 8 * case["N"], flops=rows * V * 6)
    if op == "distill":
        n = case["B"] * case["K"]
        on = n * case["masked"]
        return dict(bytes=int(2 * on * row + n * row + 5 * n + 8), flops=int(on * V * 24))
    if op == "tree":
        n = case["B"] * case["N"]
        parent = synth.tree_parents((4, 3, 2, 1), case["N"])
        inner = len(set(parent[1:].tolist()))  # leaves have no draft row
        return dict(bytes=n * row + case["B"] * inner * row + 24 * n, flops=(n + case["B"] * inner) * V * 8)
    B, K = case["B"], case["K"]
    k = (K + 1) / 2 if case["ragged"] else K
    if case["T"] == 0.0:
        return dict(bytes=int(B * (k + 1) * row + 12 * B * K), flops=int(B * (k + 1) * V))
    read = B * (2 * k + 1) * row + 21 * B * K
    flops = B * (2 * k + 1) * V * 6
    if op == "spec":
        read += 8 * B * K  # the draft rows are the verification's: read once
    if op != "verify":
        read += B * K * row + 4 * B * K + 8
        flops += (B if op in ("rejected", "spec") else B * K) * V * 24
    return dict(bytes=int(read), flops=int(flops))


def tolerance(case):
    """Tokens, lengths and masks are decided in the same arithmetic up to the
    rounding of 32-bit sums: a decision may differ only where a uniform lies
    within about 1e-7 of an edge (a token of a long flat row at the most).
    Losses are 32-bit sums (about 1e-6); gradients are rounded to the dtype of
    the logits: to 8 bits (a relative error of 1.7e-3 in bf16), or to 24 after
    32-bit exponentials of logits up to 20."""
    differ = 0.004
    if case["op"] in ("verify", "tree", "sample"):
        return {"rel": 0.0, "differ": differ}
    if case["dtype"] == "bf16":
        return {"rel": 6e-3, "max": 0.02, "differ": differ}
    return {"rel": 2e-5, "max": 1e-3, "differ": differ}


# --------------------------------------------------------------------------
# The same results in 64 bits, by torch
# --------------------------------------------------------------------------

def _draw(mass, u):
    """Smallest id whose running sum exceeds u * sum, per row."""
    c = mass.cumsum(-1)
    hit = c > (u.double() * c[:, -1]).unsqueeze(-1)
    return hit.to(torch.uint8).argmax(-1).to(torch.int32)


def _verify_exact(t, d, tokens, ua, ur, length, T):
    B, K1, _ = t.shape
    K = K1 - 1
    acc = torch.zeros(B, dtype=torch.int32, device=DEV)
    toks = torch.full((B, K + 1), -1, dtype=torch.int32, device=DEV)
    rmask = torch.zeros(B, K, dtype=torch.uint8, device=DEV)
    for b in range(B):
        kb = K if length is None else int(length[b])
        y = tokens[b, :kb].long()
        if T == 0.0:
            top = t[b, :kb + 1].double().argmax(-1)
            miss = (top[:kb] != y).nonzero()
        else:
            p = torch.softmax(t[b, :kb + 1].double() / T, -1)
            q = torch.softmax(d[b, :kb].double() / T, -1)
            at = torch.arange(kb, device=DEV)
            miss = (ua[b, :kb].double() >= p[at, y] / q[at, y]).nonzero()
        a = int(miss[0]) if miss.numel() else kb
        if T == 0.0:
            extra = top[a]
        else:
            mass = (p[a] - q[a]).clamp_min(0.0) if a < kb else p[a]
            extra = _draw(mass[None], ur[b:b + 1])[0]
        acc[b] = a
        toks[b, :a] = tokens[b, :a]
        toks[b, a] = extra
        if a < kb:
            rmask[b, a] = 1
    return acc, toks, rmask


def _distill_exact(t, d, kind, beta, tau, mask):
    B, K, V = d.shape
    rows = torch.zeros(B * K, dtype=torch.float64, device=DEV)
    grad = torch.zeros(B * K, V, dtype=torch.float64, device=DEV)
    t, d = t.reshape(B * K, V), d.reshape(B * K, V)
    on = torch.ones(B * K, dtype=torch.bool, device=DEV) if mask is None else mask.reshape(-1) != 0
    ids = on.nonzero()[:, 0]
    step = max(1, (32 << 20) // V)
    for r in range(0, ids.numel(), step):
        i = ids[r:r + step]
        lp = torch.log_softmax(t[i].double() / tau, -1)
        lq = torch.log_softmax(d[i].double() / tau, -1)
        p, q = lp.exp(), lq.exp()
        if kind == "fkl":
            rows[i] = (p * (lp - lq)).sum(-1)
            grad[i] = (q - p) / tau
        elif kind == "rkl":
            div = (q * (lq - lp)).sum(-1)
            rows[i] = div
            grad[i] = q * (lq - lp - div[:, None]) / tau
        else:
            lm = torch.log(beta * p + (1 - beta) * q)
            kq = (q * (lq - lm)).sum(-1)
            rows[i] = beta * (p * (lp - lm)).sum(-1) + (1 - beta) * kq
            grad[i] = (1 - beta) * q * (lq - lm - kq[:, None]) / tau
    total, count = rows.sum(), on.sum()
    loss = torch.stack([total / count.clamp_min(1), total])
    return loss, rows.reshape(B, K), grad.reshape(B, K, V)


def exact(case, seed):
    s = _inputs(case, seed)
    op, T = case["op"], case["T"]
    if op == "tree":
        return None  # whole numbers, which the tests compare with the library's fp64 oracle
    if op == "sample":
        mass = (1 - case["beta"]) * torch.softmax(s["q"].double() / T, -1)
        if s["p"] is not None:
            mass += case["beta"] * torch.softmax(s["p"].double() / T, -1)
        return _draw(mass, s["u"])
    if op == "distill":
        return _distill_exact(s["t"], s["d"], case["kind"], case["beta"], T, s["mask"])
    first = ()
    if op == "spec":
        q = torch.softmax(s["d"].double() / T, -1)
        s["tokens"] = torch.stack([_draw(q[:, i], s["up"][i]) for i in range(case["K"])], 1)
        first = (s["tokens"],)
    out = _verify_exact(s["t"], s["d"], s["tokens"], s["ua"], s["ur"], s["len"], T)
    if op == "verify":
        return out
    mask = None if op == "step" else out[2]
    return first + out + _distill_exact(s["t"][:, :case["K"]], s["d"], case["kind"], case["beta"], T, mask)
