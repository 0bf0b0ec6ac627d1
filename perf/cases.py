"""The performance cases of the draft-correlation path: what a serving program asks of it.

Three kinds of call:

  block   one draft block, logits to draft: `topk` and then the pass that fits the width and the
          embedding type (`score_walk` / `_certified` / `score_viterbi` for bf16 tables up to
          d = 256, else `candidate_vectors` and `pair_walk` / `_certified` / `pair_viterbi`), made as
          separate calls with kept buffers ("calls"), as one recorded graph ("graph"), or through
          `draft_block`, which allocates everything ("draft_block").
  topk    the logits pass alone (fp32 or bf16 logits, with or without the confidence features).
  scorer  the scoring-Transformer stand-in over the candidate lattice.

Sizes come from the configurations, tests and benchmark of this repository or are generic.
"""
from __future__ import annotations

import math

import torch

import paper_2608_20530_amd as L

DTYPE = {"bf16": torch.bfloat16, "fp32": torch.float32}
STD = (0.5, 2.0, 4.0)  # noise of high-, middle- and low-entropy requests
DECODES = ("greedy", "certified", "exact")


def _block(name, N, B, K, V, d, logits="bf16", table="bf16", decode="greedy", via="calls",
           anchor=False, weight=0.0, masked=0.0):
    c = {"kind": "block", "N": N, "B": B, "K": K, "V": V, "d": d, "logits": logits, "table": table,
         "decode": decode, "via": via, "anchor": anchor, "weight": weight, "masked": masked}
    return dict(c, name=name) if name else c


def _topk(name, N, B, K, V, logits="bf16", features=False):
    c = {"kind": "topk", "N": N, "B": B, "K": K, "V": V, "logits": logits, "features": features}
    return dict(c, name=name) if name else c


def _scorer(name, N, S, K, H, F, layers):
    c = {"kind": "scorer", "N": N, "S": S, "K": K, "H": H, "F": F, "layers": layers}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user, one request: latency is all that counts
        _block("block one request", 1, 16, 8, 151936, 256),
        # the smallest configuration, all fp32, replayed from its graph
        _block("block tiny graph fp32", 1, 8, 4, 32000, 64, logits="fp32", table="fp32", via="graph"),
        # a lightly loaded server that wants decisions independent of fp32 rounding
        _block("block 16 certified graph", 16, 16, 16, 151936, 256, decode="certified", via="graph"),
        # the benchmark's workload: a busy server
        _block("block 64 requests", 64, 16, 16, 151936, 256),
        # the stress workload: the largest batch, vocabulary and width
        _block("block 256 requests wide", 256, 16, 32, 262144, 512),
        # nothing is a round number: exact decode, an anchor, the drafter's log-probabilities in the
        # score, a tenth of the vocabulary banned by a grammar
        _block("block ragged exact", 23, 13, 11, 100003, 176, decode="exact", anchor=True,
               weight=0.5, masked=0.1),
        # vectors as wide as the paper's heads, exact decode
        _block("block d 1024 exact", 32, 16, 8, 151936, 1024, decode="exact"),
        # the one-call convenience on full-precision tensors and an odd vocabulary
        _block("draft_block fp32", 8, 12, 20, 32001, 192, logits="fp32", table="fp32",
               via="draft_block", anchor=True),
        # node construction's inputs from full-precision logits: candidates with their features
        _topk("topk features fp32", 48, 16, 32, 131072, logits="fp32", features=True),
        # the head's encoder for one request (the paper's widths, depth and K)
        _scorer("scorer one request", 1, 15, 8, 1024, 2048, 2),
        # the same for the benchmark's batch
        _scorer("scorer 64 requests", 64, 15, 16, 1024, 2048, 2),
        # a smaller head over an odd lattice
        _scorer("scorer ragged", 11, 9, 13, 768, 1152, 3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choices(("block", "topk", "scorer"), (6, 2, 3))[0]
        if kind == "scorer":
            S, K = rng.randint(4, 20), rng.randint(3, 16)
            c = _scorer(None, _log(rng, 1, 64), S, K, 256 * rng.randint(2, 4),
                        128 * rng.randint(6, 16), rng.randint(1, 3))
            if S * K > 256:
                continue
        else:
            N, B, K = _log(rng, 1, 256), rng.randint(4, 17), _log(rng, 2, 48)
            V, wide = _log(rng, 20000, 262144), rng.random() < 0.25
            logits = "fp32" if wide else "bf16"
            if kind == "topk":
                c = _topk(None, N, B, K, V, logits, rng.random() < 0.5)
            else:
                table = "fp32" if wide and rng.random() < 0.5 else "bf16"
                d = 16 * _log(rng, 3, 64)
                decode = rng.choice(DECODES)
                if decode == "certified" and (table == "fp32" or d > 512):
                    decode = "greedy"
                via = rng.choices(("calls", "graph", "draft_block"), (4, 2, 1))[0]
                if via == "draft_block":
                    decode = "greedy"
                c = _block(None, N, B, K, V, d, logits, table, decode, via, rng.random() < 0.4,
                           rng.choice((0.0, 0.0, 0.5)), rng.choice((0.0, 0.0, 0.1)))
        # no dearer than the largest listed case
        w = work(c)
        if w["bytes"] > 2.4e9 or w["flops"] > (1.4e11 if kind == "block" else 5.5e11):
            continue
        if kind == "block" and c["table"] == "fp32" and w["flops"] > 1e10:
            continue
        return c


# ---- inputs ---------------------------------------------------------------------------------------

def _generator(seed, tag):
    return torch.Generator(device="cuda").manual_seed((seed * 1_000_003 + tag) & ((1 << 62) - 1))


def _make_logits(c, seed):
    """Gaussian noise of the request's entropy tier, a Zipf-ranked bump on 32 ids of every slot and,
    where asked for, a share of the ids at -inf."""
    N, B, V = c["N"], c["B"], c["V"]
    g = _generator(seed, 1)
    out = torch.empty(N, B, V, dtype=DTYPE[c["logits"]], device="cuda")
    bump = 4.0 * torch.arange(1, 33, device="cuda", dtype=torch.float64).pow(-1.1).float()
    at_once = max(1, (1 << 27) // (B * V))
    for n in range(0, N, at_once):
        m = min(at_once, N - n)
        x = torch.randn(m, B, V, generator=g, device="cuda")
        x *= torch.tensor([STD[(n + i) % 3] for i in range(m)], device="cuda")[:, None, None]
        ids = torch.randint(0, V, (m, B, 32), generator=g, device="cuda")
        x.scatter_(2, ids, x.gather(2, ids) + bump)
        if c.get("masked"):
            x.masked_fill_(torch.rand(V, generator=g, device="cuda") < c["masked"], -math.inf)
        out[n:n + m] = x
    return out


def _make_head(c, seed):
    V, d, g = c["V"], c["d"], _generator(seed, 2)
    E = torch.randn(V, d, generator=g, device="cuda").mul_(0.02).to(DTYPE[c["table"]])
    W_in, W_out = (torch.randn(d, d, generator=g, device="cuda") / math.sqrt(d) for _ in range(2))
    anchor = torch.randn(c["N"], d, generator=g, device="cuda") if c["anchor"] else None
    return E, W_in, W_out, anchor


def _make_scorer(c, seed):
    N, S, K, H, F = (c[k] for k in ("N", "S", "K", "H", "F"))
    g = _generator(seed, 3)
    randn = lambda *shape: torch.randn(*shape, generator=g, device="cuda")  # noqa: E731
    X = randn(N, S * K, H)
    layers = []
    for _ in range(c["layers"]):
        w = lambda r, k: (randn(r, k) / math.sqrt(r)).to(torch.bfloat16)  # noqa: E731
        layers.append({"w_qkv": w(H, 3 * H), "w_o": w(H, H), "w_1": w(H, F), "w_2": w(F, H),
                       "g_attn": 1 + 0.1 * randn(H), "g_ffn": 1 + 0.1 * randn(H),
                       "dist_bias": 0.5 * randn(H // 128, 2 * S - 1), "same_bias": 0.5 * randn(H // 128)})
    return X, layers


# ---- one pass -------------------------------------------------------------------------------------

def _fused(c):
    return c["table"] == "bf16" and c["d"] <= 256


def prepare(case, seed):
    c = case
    if c["kind"] == "scorer":
        X, layers = _make_scorer(c, seed)
        return {"c": c, "X": X, "out": torch.empty_like(X), "packed": L.scorer_pack(layers, c["S"]),
                "workspace": L.scorer_workspace(c["N"], c["S"], c["K"], c["H"], c["F"])}
    N, B, K, V = (c[k] for k in ("N", "B", "K", "V"))
    s = {"c": c, "logits": _make_logits(c, seed)}
    if c["kind"] == "block":
        s["E"], W_in, W_out, s["anchor"] = _make_head(c, seed)
        s["packed"] = L.pack_weights(W_in, W_out)
        if c["via"] == "graph":
            s["graph"] = L.BlockGraph(s["logits"], K, s["E"], s["packed"], s["anchor"],
                                      logp_weight=c["weight"], decode=c["decode"])
            return s
        if c["via"] == "draft_block":
            return s
    new = lambda *shape, t=torch.float32: torch.empty(*shape, dtype=t, device="cuda")  # noqa: E731
    s["topk_out"] = (new(N, B, K, t=torch.int32), new(N, B, K))
    s["topk_workspace"] = L.topk_workspace(N, B, V, K)
    if c["kind"] == "topk":
        if c["features"]:
            s["topk_out"] += (new(N, B, K, 5),)
        return s
    if not _fused(c):
        s["vectors"] = (new(N, B, K, c["d"]), new(N, B, K, c["d"]))
    s["out"] = (new(N, B, t=torch.int32), new(N, B, t=torch.int32), new(N, B))
    if c["decode"] == "certified":
        s["out"] += (new(N, B, t=torch.int32),)
        s["workspace"] = L.score_walk_certified_workspace(N, B, K)
    elif c["decode"] == "exact":
        s["out"] += (new(N),)
        s["workspace"] = L.score_viterbi_workspace(N, B, K)
    else:
        s["workspace"] = L.score_walk_workspace(N, B, K)
    return s


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "scorer":
        # the forward works in place: the node states of this block are copied to where it runs
        s["out"].copy_(s["X"])
        return L.scorer_forward(s["out"], s["packed"], c["S"], c["K"], c["H"] // 128, c["F"],
                                c["layers"], workspace=s["workspace"])
    if c["kind"] == "topk":
        return L.topk(s["logits"], c["K"], out=s["topk_out"], workspace=s["topk_workspace"],
                      features=c["features"])
    third = {"greedy": None, "certified": "rescored", "exact": "score"}[c["decode"]]
    if c["via"] == "draft_block":
        return L.draft_block(s["logits"], c["K"], s["E"], s["packed"], s["anchor"],
                             logp_weight=c["weight"])
    if c["via"] == "graph":
        g = s["graph"]
        g.launch()
        r = {"ids": g.ids, "logp": g.logp, "draft": g.draft, "choice": g.choice, "logq": g.logq}
        if g.in_vec is not None:
            r["in_vec"], r["out_vec"] = g.in_vec, g.out_vec
        if third:
            r[third] = getattr(g, third)
        return r
    ids, logp = L.topk(s["logits"], c["K"], out=s["topk_out"], workspace=s["topk_workspace"])
    r = {"ids": ids, "logp": logp}
    kept = {"logp_weight": c["weight"], "out": s["out"], "workspace": s["workspace"]}
    if _fused(c):
        decode = {"greedy": L.score_walk, "certified": L.score_walk_certified,
                  "exact": L.score_viterbi}[c["decode"]]
        got = decode(ids, logp, s["E"], s["packed"], s["anchor"], **kept)
    else:
        i, o = L.candidate_vectors(ids, s["E"], s["packed"], out=s["vectors"])
        r["in_vec"], r["out_vec"] = i, o
        if c["decode"] == "certified":
            got = L.pair_walk_certified(i, o, logp, ids, s["E"], s["packed"], s["anchor"], **kept)
        else:
            decode = L.pair_walk if c["decode"] == "greedy" else L.pair_viterbi
            got = decode(i, o, logp, ids, s["anchor"], **kept)
    r["draft"], r["choice"], r["logq"] = got[:3]
    if third:
        r[third] = got[3]
    return r


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    c = case
    if c["kind"] == "scorer":
        N, S, K, H, F, n = (c[k] for k in ("N", "S", "K", "H", "F", "layers"))
        M = N * S * K
        weights = 2 * (4 * H * H + 2 * H * F)
        return {"bytes": 2 * 4 * M * H + n * weights,
                "flops": n * (2 * M * (4 * H * H + 2 * H * F) + 4 * M * S * K * H)}
    N, B, K, V = (c[k] for k in ("N", "B", "K", "V"))
    rows = N * B
    size = {"bf16": 2, "fp32": 4}
    b, f = rows * V * size[c["logits"]] + 8 * rows * K, 3 * rows * V
    if c["kind"] == "topk":
        return {"bytes": b + (20 * rows * K if c["features"] else 0), "flops": f}
    d = c["d"]
    b += min(V, rows * K) * d * size[c["table"]] + 8 * d * d + 12 * rows
    if c["via"] == "draft_block" or not _fused(c):
        b += 8 * rows * K * d  # the vectors are outputs there
    if c["via"] == "draft_block":
        b += 4 * N * (B - 1) * K * K
    if c["anchor"]:
        b += 4 * N * d
    return {"bytes": b, "flops": f + 4 * rows * K * d * d + 2 * N * (B - 1) * K * K * d}


# ---- tolerances -----------------------------------------------------------------------------------

def tolerance(case):
    """About four times the measured error against 64 bits: logp 3.5e-8 and the log-odds of the
    features as much; vectors and scores up to 6e-7 (the widest fp32 sums), logq 2.5e-7. Chosen
    indices differ only where two fp32 scores tie to within their error. The scorer rounds every
    matrix input to bf16 and a value that rounds the other way travels on: 1.8e-3 to 2.9e-3."""
    if case["kind"] == "scorer":
        return {"rel": 8e-3, "max": 0.06}
    if case["kind"] == "topk":
        return {"rel": 2e-7, "max": 5e-6}
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}


# ---- the same in 64 bits --------------------------------------------------------------------------

def _exact_topk(x, K):
    """ids by (value descending, id ascending) and log-probabilities in float64."""
    N, B, V = x.shape
    x = x.view(N * B, V)
    ids = torch.empty(N * B, K, dtype=torch.int64, device=x.device)
    logp = torch.empty(N * B, K, dtype=torch.float64, device=x.device)
    last = torch.arange(V, device=x.device).neg_() + ((1 << 32) - 1)
    step = max(1, (1 << 27) // V)
    for r in range(0, N * B, step):
        f = x[r:r + step].float() + 0.0  # -0 to +0
        bits = f.view(torch.int32).long()
        key = torch.where(bits < 0, -(bits & 0x7FFFFFFF) - 1, bits)
        top = (key * (1 << 32) + last).topk(K, dim=1).values
        ids[r:r + step] = ((1 << 32) - 1) - (top & 0xFFFFFFFF)
        v = f.double()
        logp[r:r + step] = v.gather(1, ids[r:r + step]) - v.logsumexp(1, keepdim=True)
    return ids.view(N, B, K), logp.view(N, B, K)


def _cosines(o, i):
    """sigma cos(o, i) over the last axis, a zero vector giving 0; o [..., K, d], i [..., K', d]."""
    dot = o @ i.transpose(-1, -2).contiguous()
    norm = o.norm(dim=-1)[..., :, None] * i.norm(dim=-1)[..., None, :]
    return torch.where(norm > 0, 8.0 * dot / norm.clamp_min(1e-300), torch.zeros_like(dot))


def _lowest_argmax(z):
    """Lowest index of the largest value over the last axis."""
    k = torch.arange(z.shape[-1], device=z.device).expand_as(z)
    return torch.where(z == z.amax(-1, keepdim=True), k, z.shape[-1]).amin(-1)


def _exact_block(c, seed):
    ids, logp = _exact_topk(_make_logits(c, seed), c["K"])
    E, W_in, W_out, anchor = _make_head(c, seed)
    N, B, K = ids.shape
    rows = E[ids.view(-1)].double()
    unit = []
    for W in (W_in, W_out):
        u = (rows @ W.double()).view(N, B, K, -1)
        n = u.norm(dim=-1, keepdim=True)
        unit.append(torch.where(n > 0, u / n.clamp_min(1e-300), torch.zeros_like(u)))
    i, o = unit
    S = torch.cat([_cosines(o[n:n + 8, :-1], i[n:n + 8, 1:]) for n in range(0, N, 8)])
    S0 = _cosines(anchor.double()[:, None], i[:, 0])[:, 0] if anchor is not None else None
    z0 = (S0 if S0 is not None else torch.zeros(N, K, dtype=torch.float64, device=E.device))
    w = c["weight"]
    if w:
        z0 = z0 + w * logp[:, 0]
    node = S + w * logp[:, 1:, None, :] if w else S  # [N][B-1][K][K]
    at = torch.arange(N, device=E.device)
    choice = [None] * B
    score = None
    if c["decode"] == "exact":
        best, back = z0, []
        for t in range(B - 1):
            through = (best[:, :, None] + node[:, t]).transpose(1, 2)  # [N][k][predecessor]
            back.append(_lowest_argmax(through))
            best = through.amax(-1)
        choice[B - 1] = _lowest_argmax(best)
        score = best.amax(-1)
        for t in range(B - 1, 0, -1):
            choice[t - 1] = back[t - 1][at, choice[t]]
    else:
        choice[0] = _lowest_argmax(z0)
        for t in range(1, B):
            choice[t] = _lowest_argmax(node[at, t - 1, choice[t - 1]])
    logq = []
    for t in range(B):
        z = z0 if t == 0 else node[at, t - 1, choice[t - 1]]
        logq.append(z[at, choice[t]] - z.logsumexp(-1))
    r = {"ids": None, "logp": logp, "draft": None, "choice": None, "logq": torch.stack(logq, 1)}
    if c["via"] == "draft_block" or not _fused(c):
        r["in_vec"], r["out_vec"] = i, o
    if c["via"] == "draft_block":
        r["S"], r["S0"] = S, S0
    elif c["decode"] == "exact":
        r["score"] = score
    return r


def _exact_scorer(c, seed):
    X, layers = _make_scorer(c, seed)
    N, n, H = X.shape
    heads, S = H // 128, c["S"]
    x = X.double()
    slot = torch.arange(n, device=X.device) // c["K"]
    apart = slot[:, None] - slot[None, :]
    norm = lambda v, g: v / (v.square().mean(-1, keepdim=True) + 1e-6).sqrt() * g.double()  # noqa: E731
    for p in layers:
        bias = p["dist_bias"].double()[:, apart + S - 1] + p["same_bias"].double()[:, None, None] * (apart == 0)
        qkv = norm(x, p["g_attn"]) @ p["w_qkv"].double()
        q, k, v = (t.view(N, n, heads, 128).transpose(1, 2).contiguous() for t in qkv.split(H, -1))
        a = (q @ k.transpose(-1, -2).contiguous() / math.sqrt(128) + bias).softmax(-1) @ v
        x = x + a.transpose(1, 2).reshape(N, n, H) @ p["w_o"].double()
        h = norm(x, p["g_ffn"]) @ p["w_1"].double()
        x = x + (h * h.sigmoid()) @ p["w_2"].double()
    return x


def exact(case, seed):
    c = case
    if c["kind"] == "scorer":
        return _exact_scorer(c, seed)
    if c["kind"] == "block":
        return _exact_block(c, seed)
    _, logp = _exact_topk(_make_logits(c, seed), c["K"])
    if not c["features"]:
        return None, logp
    rank = torch.arange(c["K"], device=logp.device, dtype=torch.float64).expand_as(logp)
    return None, logp, torch.stack([logp, logp.exp(), logp[..., :1] - logp, rank / max(1, c["K"] - 1),
                                    (rank == 0).double()], -1)
