"""The work a user of this library has it do, as cases to be timed.

Each case is one call (or one short chain of calls) of the public binding on a
batch of sentences: decoding one sentence, a training minibatch's loss, the
two big benchmark batches, minimum-Bayes-risk decoding of a development set,
the labelled one-stage parser, document-length sentences, and the biaffine
scorers in front of the CRF.  Lengths come from the lognormal laws of
``workloads.py`` (treebank-like), scores from N(0, sd^2) as there.

``listed()`` names the cases, ``draw(rng)`` draws another one of the same
ranges, ``prepare`` makes a case's inputs and plan, ``run`` is one pass,
``work`` what a pass cannot do without, ``tolerance`` how far another correct
implementation may be off, and ``exact`` the same outputs in float64 by plain
torch.
"""
import math

import numpy as np
import torch

from paper_2008_03736_amd import binding
from paper_2008_03736_amd import workloads

DEVICE = "cuda:0"
FORBIDDEN = workloads.FORBIDDEN

# treebank-like length laws (mean, sd, shortest, longest)
TREEBANK = dict(law="lognormal", mean=25.0, std=12.0, lo=2, hi=140)
LONGER = dict(law="lognormal", mean=28.0, std=16.0, lo=2, hi=240)


def _case(name, op, B, law, mean=0.0, std=0.0, lo=1, hi=1, sd=2.0, labels=1, d=0, forbid=0.0, pad=0, lseed=0):
    """op: the call; B sentences with lengths from (law, mean, std, lo, hi) at
    seed lseed; sd: of the scores; labels: L; d: representation size of the
    scorers; forbid: share of spans at -1e4; pad: fence posts of padding past
    the longest sentence."""
    c = dict(op=op, B=B, law=law, mean=mean, std=std, lo=lo, hi=hi, sd=sd, labels=labels, d=d, forbid=forbid,
             pad=pad, lseed=lseed)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one sentence of an interactive parser: launch and latency only
        _case("decode_one", "cky", 1, "uniform", lo=23, hi=23),
        # a small evaluation or serving batch, the `tiny` workload
        _case("parse_tiny", "parse", 32, "uniform", lo=5, hi=40, sd=1.0),
        # a training minibatch of about 5,000 words: loss of the gold trees and its gradient
        _case("loss_batch", "loss", 200, **TREEBANK),
        # the same through autograd, for a program with its own loss on log Z
        _case("logz_autograd", "logz", 300, **TREEBANK, lseed=1),
        # the benchmark batch (`mixed`): inside, marginals and decoding
        _case("parse_mixed", "parse", 5000, **TREEBANK),
        # batches with a longer tail (`longer`)
        _case("parse_longer", "parse", 2000, **LONGER),
        # minimum-Bayes-risk decoding of a development set
        _case("mbr_dev", "mbr", 1700, **TREEBANK, lseed=2),
        # one-stage labelled parser, training pass (`labeled`: L = 26)
        _case("labeled_fwd_bwd", "lfwdbwd", 1000, **TREEBANK, sd=1.0, labels=26),
        # one-stage labelled parser, decoding
        _case("labeled_decode", "lcky", 1000, **TREEBANK, sd=1.0, labels=26),
        # documents or unsplit paragraphs (`stress`): charts past one CU's LDS
        _case("parse_long", "parse", 64, "uniform", lo=256, hi=256, sd=3.0, forbid=0.05),
        # the span scorer in front of the benchmark batch, at the paper's d = 500
        _case("span_scores", "scores", 5000, **TREEBANK, d=500),
        # second stage of the two-stage parser: label scores (d = 100, a full
        # treebank label set) and the labels of decoded trees
        _case("label_stage", "labels", 100, **TREEBANK, labels=138, d=100, lseed=3),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any call above, on batches of one sentence up to the
    largest listed, short to document-length sentences, odd padding, 2 to 160
    labels, d of 32 to 500."""
    op = rng.choice(["parse", "parse", "cky", "loss", "logz", "mbr", "lfwdbwd", "lcky", "long", "long", "scores",
                     "scores", "labels"])
    lseed = rng.randrange(1 << 30)
    if op == "long":   # sentences past what one CU's LDS holds, for any unlabelled call
        hi = rng.randrange(144, 400)
        lo = rng.choice([hi, rng.randrange(20, hi)])
        most = max(1, min(64, int(64 * (256.0 / hi) ** 3)))
        return _case(None, rng.choice(["parse", "parse", "cky", "loss", "mbr"]), _log_uniform(rng, 1, most), "uniform",
                     lo=lo, hi=hi, sd=rng.choice([1.0, 2.0, 3.0]), forbid=rng.choice([0.0, 0.05]),
                     pad=rng.choice([0, 0, 3]), lseed=lseed)
    labelled = op in ("lfwdbwd", "lcky", "labels")
    B = _log_uniform(rng, 1, 1000 if labelled else 5000)
    mean = rng.uniform(8.0, 32.0)
    law = dict(law="lognormal", mean=round(mean, 2), std=round(mean * rng.uniform(0.3, 0.6), 2), lo=rng.choice([1, 2]),
               hi=rng.choice([60, 100, 140]))
    labels = d = 0
    if labelled:
        labels = _log_uniform(rng, 2, 160)
        d = 4 * rng.randrange(8, 64) if op == "labels" else 0
        # padded label scores of at most about half a gigabyte
        B = max(1, min(B, int(1.3e8 / (labels * (law["hi"] + 1) ** 2))))
    elif op == "scores":
        labels, d = 1, 4 * rng.randrange(8, 126)
    return _case(None, op, B, sd=rng.choice([1.0, 2.0]), labels=max(1, labels), d=d, pad=rng.choice([0, 0, 5]),
                 lseed=lseed, **law)


def _lengths(case):
    rng = np.random.default_rng(case["lseed"])
    if case["law"] == "uniform":
        return rng.integers(case["lo"], case["hi"] + 1, size=case["B"]).astype(np.int32)
    return workloads.lognormal_lengths(rng, case["B"], case["mean"], case["std"], case["lo"], case["hi"])


def _gold_trees(lengths, n1, seed):
    """A random binary tree per sentence, preorder rows padded with -1."""
    rng = np.random.default_rng(seed)
    R = 2 * (n1 - 1) - 1
    out = np.full((len(lengths), R, 2), -1, np.int32)
    for b, n in enumerate(lengths):
        rows, todo, u = [], [(0, int(n))], rng.random(int(n))
        while todo:
            i, j = todo.pop()
            rows.append((i, j))
            if j - i >= 2:
                k = i + 1 + int(u[i] * (j - i - 1))
                todo.append((k, j))
                todo.append((i, k))
        out[b, :len(rows)] = rows
    return torch.from_numpy(out).to(DEVICE)


def _inputs(case, seed):
    """The case's inputs on the GPU, from the seed alone."""
    lengths = _lengths(case)
    B, n1, L, d = case["B"], int(lengths.max()) + 1 + case["pad"], case["labels"], case["d"]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEVICE)

    x = dict(lengths=lengths, n1=n1)
    if case["op"] in ("scores", "labels"):
        def bf16(t):
            return t.to(torch.bfloat16).view(torch.int16)
        x["rl"], x["rr"] = bf16(normal(B, n1, d)), bf16(normal(B, n1, d))
        ldw = (d + 1 + 7) // 8 * 8
        x["w"] = bf16(normal(L, d, ldw) * (2.0 / d))
    else:
        shape = (B, n1, n1) if L == 1 else (B, n1, n1, L)
        x["scores"] = normal(*shape).mul_(case["sd"])
        if case["forbid"] > 0:
            hit = torch.rand((B, n1, n1), generator=g, device=DEVICE) < case["forbid"]
            x["scores"][hit] = FORBIDDEN
    if case["op"] in ("loss", "labels"):
        x["gold"] = _gold_trees(lengths, n1, seed)
    if case["op"] == "logz":
        x["upstream"] = normal(B)
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s["op"] = case["op"]
    L = 1 if case["op"] in ("scores", "labels") else case["labels"]
    s["plan"] = binding.Plan(s["lengths"], n1=s["n1"], num_labels=L, device=DEVICE)
    # Outputs a program keeps across batches of one shape.  A training step
    # (loss, logz) takes fresh gradients instead.
    B, n1 = case["B"], s["n1"]
    R = 2 * (n1 - 1) - 1

    def f32(*shape):
        return torch.zeros(shape, dtype=torch.float32, device=DEVICE)

    def i32(*shape):
        return torch.zeros(shape, dtype=torch.int32, device=DEVICE)

    op = case["op"]
    if op in ("parse", "mbr"):
        s["out"] = dict(logZ=f32(B), marginals=f32(B, n1, n1), spans=i32(B, R, 2), best=f32(B))
    elif op == "cky":
        s["out"] = dict(spans=i32(B, R, 2), best=f32(B))
    elif op == "lfwdbwd":
        s["out"] = dict(logZ=f32(B), marginals=f32(B, n1, n1, L))
    elif op == "lcky":
        s["out"] = dict(spans=i32(B, R, 2), labels=i32(B, R), best=f32(B))
    elif op == "scores":
        s["out"] = dict(scores=f32(B, n1, n1))
    elif op == "labels":
        s["out"] = dict(scores=f32(B, n1, n1, case["labels"]) if case["labels"] > 1 else f32(B, n1, n1))
        s["labels"] = i32(B, R)
    elif op == "logz":
        s["scores"].requires_grad_(True)
    return s


def run(s):
    op, plan = s["op"], s["plan"]
    if op == "parse":
        return plan.parse(s["scores"], **s["out"])
    if op == "mbr":
        return plan.mbr_decode(s["scores"], **s["out"])
    if op == "cky":
        return plan.cky_decode(s["scores"], **s["out"])
    if op == "loss":
        return plan.gold_loss(s["scores"], s["gold"])
    if op == "logz":
        logz = binding.log_partition(s["scores"], plan)
        grad, = torch.autograd.grad(logz, s["scores"], s["upstream"])
        return logz.detach(), grad
    if op == "lfwdbwd":
        return plan.inside_fwd_bwd(s["scores"], **s["out"])
    if op == "lcky":
        return plan.cky_decode_labeled(s["scores"], **s["out"])
    scores = plan.biaffine_scores(s["rl"], s["rr"], s["w"], **s["out"])
    if op == "scores":
        return scores
    B, n1 = scores.shape[:2]
    labels = plan.label_spans(scores.view(B, n1, n1, -1), s["gold"], labels=s["labels"])
    return scores, labels


def work(case):
    """Bytes: each valid score, representation and weight read once, each
    valid output written once.  Operations: a multiply and an add per split
    point for the inside and for each of the split's two outside terms, an
    add and a compare per split point for CKY, an exponential and two more per label, and the
    scorer's two products."""
    n = _lengths(case).astype(np.int64)
    B, op, L, d = case["B"], case["op"], case["labels"], case["d"]
    T = int(((n + 1) * n * (n - 1) // 6).sum())       # split points
    P = int((n * (n + 1) // 2).sum())                 # spans
    rows = int((2 * n - 1).sum())                     # tree nodes
    if op == "parse" or op == "mbr":
        return dict(bytes=8 * P + 8 * rows + 8 * B, flops=8 * T)
    if op == "cky":
        return dict(bytes=4 * P + 8 * rows + 4 * B, flops=2 * T)
    if op == "loss":
        return dict(bytes=8 * P + 8 * rows + 4 * B, flops=6 * T)
    if op == "logz":
        return dict(bytes=8 * P + 8 * B, flops=6 * T)
    if op == "lfwdbwd":
        return dict(bytes=8 * P * L + 4 * B, flops=6 * T + 6 * P * L)
    if op == "lcky":
        return dict(bytes=4 * P * L + 12 * rows + 4 * B, flops=2 * T + P * L)
    # n + 1 fence posts each way; W; the valid cells
    by = 4 * int((n + 1).sum()) * d + 2 * L * d * (d + 1) + 4 * P * L
    fl = L * int((2 * n * (d + 1) * d + d * n * (n + 1)).sum())
    if op == "labels":
        by += 8 * rows + 4 * rows + 4 * rows * L   # the spans, their labels, the label scores at the spans
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """Decoded trees, their labels and scores come from float64 charts (or
    exact float32 maxima) and must be the same.  The rest is float32: against
    ``exact`` log Z is off by 3e-8, marginals by 3e-7 on treebank lengths and
    1.2e-6 at 256 words (largest 1.2e-5), the scorer (its inner product held
    in 16 bits of mantissa) by 2.5e-6 (largest 7e-5); about four times these,
    and room for the few near-ties of trees over marginals and of labels."""
    op = case["op"]
    if op in ("cky", "lcky"):
        return "exact"
    if op == "scores":
        return {"rel": 1e-5, "max": 4e-4}
    if op == "labels":
        return {"rel": 1e-5, "max": 4e-4, "differ": 1e-3}
    if op == "mbr":
        return {"rel": 5e-6, "max": 1e-4, "differ": 2e-3}
    return {"rel": 5e-6, "max": 1e-4}


# ---------------------------------------------------------------------------
# The same outputs in float64.


def _diagonals(sc, N, lengths):
    """Scores [b, N+1, N+1] float64 by (width, start), -inf off the sentence."""
    b = sc.shape[0]
    D = torch.full((b, N + 1, N + 1), -math.inf, dtype=torch.float64, device=sc.device)
    start = torch.arange(N + 1, device=sc.device)
    for w in range(1, N + 1):
        diag = sc.diagonal(w, 1, 2)[:, :N + 1 - w]
        ok = start[None, :N + 1 - w] + w <= lengths[:, None]
        D[:, w, :N + 1 - w] = torch.where(ok, diag, -math.inf)
    return D


def _by_end(D, N):
    """(width, start) -> (width, end)."""
    E = torch.full_like(D, -math.inf)
    for w in range(1, N + 1):
        E[:, w, w:] = D[:, w, :N + 1 - w]
    return E


def _chunks(lengths, n1):
    """Sentence ids sorted by length, in groups of a bounded chart size."""
    order = np.argsort(lengths, kind="stable")
    a = 0
    while a < len(order):
        e = a
        while e < len(order) and (e + 1 - a) * (int(lengths[order[e]]) + 2) ** 2 <= 4_000_000:
            e += 1
        e = max(e, a + 1)
        yield torch.from_numpy(order[a:e].copy()).to(DEVICE), int(lengths[order[e - 1]])
        a = e


def _inside_outside(scores, lengths):
    """log Z [B] and span marginals [B, N1, N1], float64."""
    B, n1 = scores.shape[:2]
    lens = torch.from_numpy(lengths.astype(np.int64)).to(DEVICE)
    logZ = torch.empty(B, dtype=torch.float64, device=DEVICE)
    marg = torch.zeros((B, n1, n1), dtype=torch.float64, device=DEVICE)
    for ids, N in _chunks(lengths, n1):
        ln = lens[ids]
        S = _diagonals(scores[ids, :N + 1, :N + 1].double(), N, ln)
        A, E = torch.full_like(S, -math.inf), torch.full_like(S, -math.inf)   # alpha by start, by end
        A[:, 1], E[:, 1, 1:] = S[:, 1], S[:, 1, :N]
        for w in range(2, N + 1):
            m = N + 1 - w
            a = torch.logsumexp(A[:, 1:w, :m] + E[:, 1:w, w:].flip(1), 1) + S[:, w, :m]
            A[:, w, :m] = a
            E[:, w, w:] = a
        z = A[torch.arange(len(ids), device=DEVICE), ln, 0]
        OS, OE = torch.full_like(S, -math.inf), torch.full_like(S, -math.inf)  # outside + own score
        for v in range(N, 0, -1):
            m = N + 1 - v
            o = torch.full((len(ids), m), -math.inf, dtype=torch.float64, device=DEVICE)
            if v < N:
                left = OE[:, v + 1:, v:] + E[:, 1:m, :m]
                right = OS[:, v + 1:, :m] + A[:, 1:m, v:]
                o = torch.logsumexp(torch.cat([left, right], 1), 1)
            o[:, 0] = torch.where(ln == v, 0.0, o[:, 0])
            so = o + S[:, v, :m]
            OS[:, v, :m] = so
            OE[:, v, v:] = so
            p = torch.exp(A[:, v, :m] + o - z[:, None])
            p = torch.where(torch.isfinite(S[:, v, :m]), p, 0.0)
            i = torch.arange(m, device=DEVICE)
            marg[ids[:, None], i[None], i[None] + v] = p
        logZ[ids] = z
    return logZ, marg


def _cky(scores, lengths):
    """Best trees [B, R, 2] (preorder, -1 past the tree) and their scores."""
    B, n1 = scores.shape[:2]
    lens = torch.from_numpy(lengths.astype(np.int64)).to(DEVICE)
    R = 2 * (n1 - 1) - 1
    spans = torch.full((B, R, 2), -1, dtype=torch.int64, device=DEVICE)
    best = torch.empty(B, dtype=torch.float64, device=DEVICE)
    for ids, N in _chunks(lengths, n1):
        ln, b = lens[ids], len(ids)
        S = _diagonals(scores[ids, :N + 1, :N + 1].double(), N, ln)
        A, E = torch.full_like(S, -math.inf), torch.full_like(S, -math.inf)
        K = torch.zeros(S.shape, dtype=torch.int64, device=DEVICE)
        A[:, 1], E[:, 1, 1:] = S[:, 1], S[:, 1, :N]
        for w in range(2, N + 1):
            m = N + 1 - w
            v, k = (A[:, 1:w, :m] + E[:, 1:w, w:].flip(1)).max(1)
            A[:, w, :m] = v + S[:, w, :m]
            E[:, w, w:] = A[:, w, :m]
            K[:, w, :m] = k + 1
        at = torch.arange(b, device=DEVICE)
        best[ids] = A[at, ln, 0]
        # preorder walk of all trees at once, a stack of right children each
        stack = torch.zeros((b, N + 2, 2), dtype=torch.int64, device=DEVICE)
        top = torch.zeros(b, dtype=torch.int64, device=DEVICE)
        i, j = torch.zeros_like(ln), ln.clone()
        for r in range(2 * N - 1):
            live = r < 2 * ln - 1
            row = torch.stack([i, j], 1)
            spans[ids, r] = torch.where(live[:, None], row, -1)
            w = (j - i).clamp(min=0)
            k = i + K[at, w, i.clamp(max=N)]
            inner = live & (w >= 2)
            push = torch.stack([k, j], 1)
            stack[at, top] = torch.where(inner[:, None], push, stack[at, top])
            top = top + inner.long()
            leaf = live & (w < 2) & (top > 0)
            top = top - leaf.long()
            pop = stack[at, top]
            i = torch.where(leaf, pop[:, 0], i)
            j = torch.where(inner, k, torch.where(leaf, pop[:, 1], j))
    return spans, best


def _valid(lengths, n1):
    return torch.from_numpy(workloads.valid_mask(lengths, n1)).to(DEVICE)


def exact(case, seed):
    x = _inputs(case, seed)
    op, lengths, n1 = case["op"], x["lengths"], x["n1"]
    if op in ("parse", "mbr", "loss", "logz"):
        logZ, mu = _inside_outside(x["scores"], lengths)
        if op == "parse":
            return (logZ, mu, *_cky(x["scores"], lengths))
        if op == "mbr":
            return (logZ, mu, *_cky(mu, lengths))
        if op == "logz":
            return logZ, mu * x["upstream"].double()[:, None, None]
        g = x["gold"].long()
        ok = g[..., 0] >= 0
        b, r = ok.nonzero(as_tuple=True)
        i, j = g[b, r, 0], g[b, r, 1]
        loss = logZ.clone()
        loss.index_add_(0, b, -x["scores"][b, i, j].double())
        mu[b, i, j] -= 1.0
        return loss, mu
    if op == "cky":
        return _cky(x["scores"], lengths)
    if op == "lfwdbwd":
        s4 = x["scores"].double()
        s = torch.logsumexp(s4, 3)
        logZ, mu = _inside_outside(s, lengths)
        return logZ, mu[..., None] * torch.exp(s4 - s[..., None])
    if op == "lcky":
        top = x["scores"].max(3).values
        spans, best = _cky(top, lengths)
        b = torch.arange(len(lengths), device=DEVICE)[:, None]
        i, j = spans.clamp(min=0).unbind(2)
        lab = x["scores"][b, i, j].argmax(2)
        return spans, torch.where(spans[..., 0] >= 0, lab, -1), best
    rl, rr, w = (x[k].view(torch.bfloat16).double() for k in ("rl", "rr", "w"))
    B, d, L = len(lengths), case["d"], case["labels"]
    valid = _valid(lengths, n1)
    out = torch.zeros((B, n1, n1, L), dtype=torch.float64, device=DEVICE)
    one = torch.cat([rl, torch.ones_like(rl[..., :1])], 2).reshape(B * n1, d + 1)
    rrt = rr.transpose(1, 2).contiguous()
    for q in range(L):
        u = (one @ w[q, :, :d + 1].t().contiguous()).view(B, n1, d)
        out[..., q] = torch.where(valid, torch.bmm(u, rrt), 0.0)
    if op == "scores":
        return out[..., 0]
    g = x["gold"].long()
    b = torch.arange(B, device=DEVICE)[:, None]
    i, j = g.clamp(min=0).unbind(2)
    lab = torch.where(g[..., 0] >= 0, out[b, i, j].argmax(2), -1)
    return (out if L > 1 else out[..., 0]), lab
