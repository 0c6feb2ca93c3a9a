"""What a user of this library has it do, as cases that can be timed and checked.

One pass is one draft phase on logits that are resident on the GPU: reset, max_depth x expand_layer, and the
emission of the tree (finalize_tree, or finalize_tree_reranked for contexts that rerank).  The draft model's forward
passes, which a real program runs between the layers, are not part of it: layer l's logits are ready when the pass
begins, as in the benchmark.

A case's sizes: B sequences, V vocabulary, F frontier nodes and K children per node, D layers, N nodes a tree may
hold, h classifier width; dtype of the logits; top_m > 0: entropy over the M most probable tokens; rerank > 0: that
many nodes emitted by the reranking; mask: share of the vocabulary that every row of a sequence has masked (-inf).

Inputs.  A logits row is Gaussian noise of a scale of its own (sigma in 1 .. 6) on a Zipf-shaped bias over a permutation
of the token ids that the sequence's rows share; one row in twenty gets one token raised by 20.  The classifier has
the form that training gives it: its confidence grows with the joint probability of the path over several decades
(a sum of hinges at log-spaced thresholds) and falls a little with entropy and depth; so trees of rows that are sharp
grow until their budget is used up, and those of flat rows stop early.
"""
import math

import torch

from paper_2502_13652_amd import C2TContext

ZIPF, SIGMA, SPIKED = 1.05, (1.0, 6.0), 0.05
LIVE = (1.0, 1.0, 0.98, 0.98, 0.85, 0.5, 0.25, 0.1)   # share of a full frontier that is live in each layer, on average over such inputs (beta > 0)
LAYER_BYTES = 13 << 30   # logits of one phase kept apart, at most; layers past them use the first ones' again


def _case(name, B, V, F, K, D, N, h, beta, dtype="bf16", top_m=0, rerank=0, mask=0.0):
    return dict(name=name, B=B, V=V, F=F, K=K, D=D, N=N, h=h, beta=beta, dtype=dtype, top_m=top_m, rerank=rerank, mask=mask)


def listed():
    return [
        # one user's chat with a 32k vocabulary: the smallest call, where latency and launches count
        _case("one_32k", 1, 32000, 10, 10, 8, 60, 12, 0.5),
        # the same from a draft head that leaves its logits in fp32
        _case("one_32k_f32", 1, 32000, 10, 10, 6, 60, 12, 0.5, dtype="f32"),
        # one user's chat with a 128k vocabulary
        _case("one_128k", 1, 128256, 16, 16, 8, 96, 32, 0.4),
        # batched serving: 64 users, 128k vocabulary
        _case("batch64_128k", 64, 128256, 16, 16, 6, 64, 32, 0.4),
        # the largest: 256 users, 152k vocabulary, wide frontiers
        _case("batch256_152k", 256, 152064, 32, 32, 8, 128, 64, 0.3),
        # chain drafting (one child per node) for many users at once
        _case("chain1024_32k", 1024, 32000, 1, 1, 8, 8, 12, 0.5),
        # the entropy feature over the 1000 most probable tokens
        _case("batch32_top1000", 32, 128256, 16, 16, 6, 64, 32, 0.4, top_m=1000),
        # every candidate reranked at the end, nothing pruned by confidence on the way
        _case("batch32_rerank", 32, 32000, 10, 10, 6, 60, 12, 0.0, rerank=60),
        # constrained decoding: a third of the vocabulary is masked
        _case("batch16_masked", 16, 128256, 16, 16, 6, 64, 32, 0.4, mask=0.3),
        # batched serving with fp32 logits
        _case("batch32_f32", 32, 32000, 10, 10, 6, 60, 12, 0.5, dtype="f32"),
        # a few users, fp32, an odd vocabulary and classifier width
        _case("batch5_65541_f32", 5, 65541, 8, 8, 5, 40, 7, 0.3, dtype="f32"),
        # few but wide and deep trees over an odd vocabulary, the largest tree, frontier and classifier there are
        _case("wide4_20011", 4, 20011, 64, 32, 17, 1024, 256, 0.2),
    ]


def _rows(case):
    """Rows of each layer while every frontier is full: the root, then what the second pruning and the budget leave."""
    rows, nodes, live = [], 0, 1
    for _ in range(case["D"]):
        rows.append(live)
        live = min(case["F"], live * case["K"], case["N"] - nodes)
        nodes += live
    return rows


def _esz(case):
    return 4 if case["dtype"] == "f32" else 2


def _row_bytes(case):
    return case["V"] * _esz(case)


def _mean_rows(case):
    return case["B"] * sum(r * (1.0 if case["beta"] == 0 else LIVE[l] if l < len(LIVE) else 0.03) for l, r in enumerate(_rows(case)))


def draw(rng):
    def logint(lo, hi):
        return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))

    kind = rng.choice(["one", "one_f32", "batch", "batch", "batch", "batch_f32", "chain", "wide"])
    V = logint(8000, 152064)
    if rng.random() < 0.4:
        V = V // 64 * 64
    F, K, D = logint(4, 32), logint(4, 32), rng.randint(3, 8)
    B = {"one": 1, "one_f32": 1, "batch": logint(2, 256), "batch_f32": logint(2, 64), "chain": logint(64, 1024), "wide": logint(1, 8)}[kind]
    if kind == "chain":
        F, K, N = 1, 1, D
    elif kind == "wide":
        F, K, D = rng.randint(33, 64), rng.randint(16, 32), rng.randint(4, 17)
        N = min(1024, F * D)
    else:
        N = rng.randint(2 * F, 5 * F)
    c = _case("", B, V, F, K, D, N, logint(4, 256 if kind == "wide" else 64), rng.choice([0.0, 0.2, 0.3, 0.4, 0.5]),
              dtype="f32" if kind.endswith("f32") else "bf16", top_m=1000 if rng.random() < 0.2 else 0,
              mask=rng.choice([0.01, 0.3, 0.9]) if rng.random() < 0.15 else 0.0)
    if kind != "chain" and rng.random() < 0.2 and D * F * K <= 32768:
        c["rerank"] = min(1024, N)
    while c["B"] > 1 and _mean_rows(c) * _row_bytes(c) > 3e9:
        c["B"] -= 1
    del c["name"]
    return c


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed % (1 << 62))
    return g


def _classifier(case, g):
    """W1 [h][3] (P, H, d), b1, w2, b2: relu(1 - P/t_j) at log-spaced thresholds t_j, two units on entropy and depth where there is room."""
    h = case["h"]
    extra = 2 if h >= 4 else 0
    n = h - extra
    t = torch.logspace(math.log10(0.5), -6.0, n, dtype=torch.float64)
    noise = torch.randn((h, 6), generator=g, device="cuda").cpu().double()
    W1, b1, w2 = torch.zeros(h, 3, dtype=torch.float64), torch.zeros(h, dtype=torch.float64), torch.zeros(h, dtype=torch.float64)
    W1[:n, 0] = -1.0 / t
    b1[:n] = 1.0
    w2[:n] = -6.0 / n * (1.0 + 0.05 * noise[:n, 4])
    W1[:n, 1], W1[:n, 2] = 0.01 * noise[:n, 1].abs(), 0.01 * noise[:n, 2].abs()
    if extra:
        W1[n, 1], W1[n + 1, 2] = 1.0, 1.0
        w2[n], w2[n + 1] = -0.05, -0.05
    b2 = 3.0 + 0.1 * float(noise[0, 5])
    return W1.float().numpy(), b1.float().numpy(), w2.float().numpy(), float(torch.tensor(b2, dtype=torch.float32))


def _logits(case, g):
    """One tensor [B][F][stride] a layer, the stride padded to 16 bytes (what lies in the padding must not matter)."""
    B, V, F, D = case["B"], case["V"], case["F"], case["D"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    per = 16 // _esz(case)
    stride = (V + per - 1) // per * per
    apart = max(1, min(D, LAYER_BYTES // (B * F * stride * _esz(case))))
    step = max(1, (1 << 28) // (F * V))                     # sequences made at once
    layers = [torch.full((B, F, stride), 100.0, dtype=dtype, device="cuda") for _ in range(apart)]
    for b0 in range(0, B, step):
        n = min(step, B - b0)
        rank = torch.rand((n, V), generator=g, device="cuda").argsort(1)
        bias = -ZIPF * torch.log((rank + 1).float())
        if case["mask"] > 0:
            bias.masked_fill_(torch.rand((n, V), generator=g, device="cuda") < case["mask"], -math.inf)
        for x in layers:
            sigma = SIGMA[0] + (SIGMA[1] - SIGMA[0]) * torch.rand((n, F, 1), generator=g, device="cuda")
            r = torch.randn((n, F, V), generator=g, device="cuda").mul_(sigma).add_(bias[:, None])
            raised = torch.where(torch.rand((n, F, 1), generator=g, device="cuda") < SPIKED, 20.0, 0.0)
            r.scatter_add_(2, torch.randint(0, V, (n, F, 1), generator=g, device="cuda"), raised)
            x[b0:b0 + n, :, :V] = r
    return [layers[i % apart] for i in range(D)]


def _inputs(case, seed):
    g = _generator(seed)
    return _classifier(case, g), _logits(case, g)


def prepare(case, seed):
    cls, layers = _inputs(case, seed)
    ctx = C2TContext(case["B"], case["V"], case["F"], case["K"], case["D"], case["N"], case["h"], case["dtype"], case["beta"],
                     entropy_top_m=case["top_m"], rerank=1 if case["rerank"] else 0)
    ctx.set_classifier(*cls)
    return dict(ctx=ctx, layers=layers, rerank=case["rerank"], out=ctx.new_tree_out(case["rerank"] or None))


def run(state):
    ctx = state["ctx"]
    ctx.reset()
    for x in state["layers"]:
        ctx.expand_layer(x)
    if state["rerank"]:
        return ctx.finalize_tree_reranked(state["rerank"], state["out"])
    return ctx.finalize_tree(state["out"])


def work(case):
    """Every live row (their number is an average) read once and the tree written once; per logit an exponential and the sums (four operations),
    per candidate the classifier."""
    rows, n_out = _mean_rows(case), case["rerank"] or case["N"]
    written = case["B"] * (n_out * n_out + 24 * n_out + 8)
    return {"bytes": rows * _row_bytes(case) + written, "flops": 4.0 * rows * case["V"] + 10.0 * rows * case["K"] * case["h"]}


def tolerance(case):
    """Which nodes a tree holds, and their order, is decided by the definition's fp32 arithmetic on features that are
    64-bit results rounded once; so trees are the same, and what is left is the rounding of an fp32 result and of the
    sigmoid."""
    return {"rel": 1e-6, "max": 1e-5}


# ---- the definition in 64 bits ---------------------------------------------------------------------------------

def _order(x):
    """int64 keys of fp32 values that order as (value desc -> key desc), -0 as +0."""
    u = (x.float() + 0.0).view(torch.int32).long()
    return torch.where(u < 0, -1 - (u & 0x7FFFFFFF), u)


def _row_features(x, K, top_m):
    """ids [R][K], p [R][K] and H [R] of rows x [R][V], in 64 bits; equal logits by token id."""
    V = x.shape[1]
    ids = torch.arange(V, device=x.device)
    key = (_order(x) << 32) | (0xFFFFFFFF - ids)
    top = 0xFFFFFFFF - (key.topk(K, 1).values & 0xFFFFFFFF)
    del key
    xd = x.double()
    t = xd - xd.amax(1, keepdim=True)
    e = t.exp()
    Z = e.sum(1, keepdim=True)
    p = e.gather(1, top) / Z
    if top_m and top_m < V:
        t = t.topk(top_m, 1).values
        e = t.exp()
    plnp = torch.where(e > 0, (t - Z.log()) * (e / Z), 0.0)
    return top, p, -plnp.sum(1)


def _confidence(cls, P, H, d, single):
    """The classifier's logit: in fp32 (a chain of fused multiply-adds, hidden units ascending), or in 64 bits."""
    W1, b1, w2, b2 = cls
    rnd = (lambda v: v.float().double()) if single else (lambda v: v)
    z = torch.full_like(P, float(b2))
    for j in range(len(b1)):
        a = rnd(float(W1[j, 0]) * P + float(b1[j]))
        a = rnd(float(W1[j, 1]) * H + a)
        a = rnd(float(W1[j, 2]) * d + a)
        z = rnd(float(w2[j]) * a.clamp_min(0.0) + z)
    return z


def exact(case, seed):
    B, V, F, K, D, N = (case[k] for k in ("B", "V", "F", "K", "D", "N"))
    cls, layers = _inputs(case, seed)
    dev, f64 = "cuda", torch.float64
    beta = float(torch.tensor(case["beta"], dtype=torch.float32))      # the threshold arrives as an fp32
    z_beta = float(torch.tensor(math.log(beta / (1.0 - beta)), dtype=torch.float32)) if beta > 0 else -math.inf
    n_out = case["rerank"] or N
    nf = torch.ones(B, dtype=torch.long, device=dev)        # frontier sizes, and per slot: P in fp32 and 64 bits, smallest z on the path
    fP32 = torch.ones(B, F, dtype=f64, device=dev)
    fP64, fs = fP32.clone(), torch.full((B, F), math.inf, dtype=f64, device=dev)
    nodes = torch.zeros(B, dtype=torch.long, device=dev)
    tree = torch.zeros(3, B, N + 1, dtype=f64, device=dev)  # conf, joint_prob, entropy; slot N takes what is not kept
    history = []
    slot = torch.arange(F, device=dev)
    for l in range(D):
        b_of, f_of = (slot[None] < nf[:, None]).nonzero(as_tuple=True)
        tok = torch.zeros(B, F, K, dtype=torch.long, device=dev)
        p = torch.zeros(B, F, K, dtype=f64, device=dev)
        H = torch.zeros(B, F, dtype=f64, device=dev)
        step = max(1, (1 << 28) // V)
        for i in range(0, len(b_of), step):
            b, f = b_of[i:i + step], f_of[i:i + step]
            tok[b, f], p[b, f], H[b, f] = _row_features(layers[l][b, f, :V], K, case["top_m"])
        valid = (slot[None] < nf[:, None])[:, :, None].expand(B, F, K)
        P32 = (fP32[:, :, None].float() * p.float()).double()
        P64 = fP64[:, :, None] * p
        H3 = H[:, :, None].expand(B, F, K)
        z32 = _confidence(cls, P32, H3.float().double(), float(l), True)
        z64 = _confidence(cls, P64, H3, float(l), False)
        s = torch.minimum(fs[:, :, None], z32)
        if case["rerank"]:
            history.append((torch.where(valid, s, -math.inf).reshape(B, -1), z64.reshape(B, -1), P64.reshape(B, -1), H3.reshape(B, -1)))
        # first pruning, then the best by (z desc, token asc, candidate asc) within width and budget
        keep = valid & (z32 > z_beta)
        zk = torch.where(keep, z32, -math.inf).reshape(B, F * K)
        by = tok.reshape(B, F * K).argsort(dim=1, stable=True)
        by = by.gather(1, zk.gather(1, by).argsort(dim=1, descending=True, stable=True))[:, :F]
        width = by.shape[1]
        n_keep = torch.minimum(keep.reshape(B, -1).sum(1), (N - nodes).clamp(0, F))
        kept = slot[None, :width] < n_keep[:, None]
        at = torch.where(kept, nodes[:, None] + slot[None, :width], N)
        for k, v in enumerate((torch.sigmoid(z64), P64, H3)):
            tree[k].scatter_(1, at, v.reshape(B, -1).gather(1, by))
        pad = (0, F - width)
        fP32, fP64, fs = (torch.nn.functional.pad(v.reshape(B, -1).gather(1, by), pad) for v in (P32, P64, s))
        nodes, nf = nodes + n_keep, n_keep
    if case["rerank"]:
        s, z64, P64, H64 = (torch.cat(v, 1) for v in zip(*history))
        by = s.argsort(dim=1, descending=True, stable=True)[:, :n_out]
        ok = s.gather(1, by) > -math.inf
        tree = torch.stack([torch.where(ok, v.gather(1, by), 0.0) for v in (torch.sigmoid(z64), P64, H64)])
        tree = torch.nn.functional.pad(tree, (0, n_out - tree.shape[2]))
    else:
        tree = tree[:, :, :N]
    whole = {k: None for k in ("tokens", "parent", "position", "n_nodes", "mask", "status")}
    return dict(whole, conf=tree[0].contiguous(), joint_prob=tree[1].contiguous(), entropy=tree[2].contiguous())
