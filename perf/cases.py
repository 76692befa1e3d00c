"""The measured work of this framework, one pass per case through its public entry points.

A case is a dict of plain values. Its `kind` names the calls that a pass makes:

  round    Round.run: a whole verification round of a serving loop (evaluation of every drafter,
           expected accepted lengths, losses, Hedge and NormalHedge), with buffers and learner
           state built once, as a server keeps them;
  eval     eval_alpha with every output (alpha, agreement and the argmax tokens), the call of a
           program that keeps its own learner;
  topl     eval_topl with every output: EAGLE's greedy tree, L children per node;
  pruned   softmax_stats of the target's rows, then candidate_mass on the kept children: EAGLE-2's
           dynamic pruning after its children are known;
  stats    softmax_stats of a plain [rows][ld] matrix;
  feedback delayed_update, play and RegretState.update: the token-level game between two
           evaluations.

Logits follow the repository's generator: target ~ N(0, sigma^2) with a few boosted tokens per
row, drafter i = target + N(0, s_i^2) with s_i log-spaced and rotated from query to query, so
that each drafter is the best for some queries. Vocabularies run from 30000 to 152000 tokens,
odd ones among them (rows are padded to whole 16-byte vectors).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_20064_amd as hs

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
LOSSES = {"length": hs.LOSS_LENGTH, "token": hs.LOSS_ACCEPT_TOKEN, "chunk": hs.LOSS_ACCEPT_CHUNK}
MAX_BYTES = 5_300_000_000  # logits of the largest case


# ---- the cases ---------------------------------------------------------------------------------

def listed():
    return [
        # the smallest round in use: one query, a small pool, a 32000-token head in fp32, one
        # learner update per token; all latency
        dict(name="round_tiny_f32", kind="round", B=1, N=4, K=4, V=32000, dtype="f32", T=1.0,
             mode="sample", loss="token", tree=False),
        # interactive decoding: one query, eight drafters, a full chunk, a 152k-token head
        dict(name="round_single_bf16", kind="round", B=1, N=8, K=8, V=151936, dtype="bf16", T=1.0,
             mode="sample", loss="length", tree=False),
        # batched serving at a sampling temperature
        dict(name="round_batch_bf16", kind="round", B=64, N=8, K=6, V=128256, dtype="bf16", T=0.7,
             mode="sample", loss="length", tree=False),
        # the same server decoding greedily: argmax agreement instead of probabilities
        dict(name="greedy_batch_bf16", kind="round", B=64, N=8, K=6, V=128256, dtype="bf16", T=1.0,
             mode="greedy", loss="length", tree=False),
        # many small fp32 queries in one call
        dict(name="round_many_f32", kind="round", B=64, N=4, K=4, V=32000, dtype="f32", T=1.0,
             mode="sample", loss="token", tree=False),
        # a 64-node draft tree per query
        dict(name="round_tree_bf16", kind="round", B=16, N=16, K=64, V=151936, dtype="bf16", T=1.0,
             mode="sample", loss="length", tree=True),
        # the largest pool the library takes, one round of a long stream
        dict(name="round_pool_bf16", kind="round", B=32, N=64, K=8, V=151936, dtype="bf16", T=1.0,
             mode="sample", loss="length", tree=False),
        # ragged on every side: odd counts, an odd vocabulary, fp16, every output at once
        dict(name="eval_ragged_f16", kind="eval", B=13, N=5, K=7, V=50257, dtype="f16", T=0.5),
        # EAGLE's greedy tree for one query, and for the largest pool
        dict(name="topl_single_bf16", kind="topl", B=1, N=8, K=8, V=151936, dtype="bf16", T=1.0,
             L=10),
        dict(name="topl_pool_bf16", kind="topl", B=32, N=64, K=8, V=151936, dtype="bf16", T=1.0,
             L=10),
        # EAGLE-2's pruned tree for a batch: normalisers of the target's rows, then the mass
        dict(name="pruned_batch_bf16", kind="pruned", B=64, N=8, K=6, V=128256, dtype="bf16",
             T=0.7, L=10),
        # the learners between two evaluations of the largest pool
        dict(name="feedback_pool", kind="feedback", B=32, N=64, K=8),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "round", "eval", "topl", "topl", "pruned",
                       "stats", "feedback"])
    if kind == "feedback":
        return dict(kind=kind, B=_logint(rng, 1, 256), N=rng.randint(2, 64), K=rng.randint(2, 16))
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    V = _logint(rng, 30000, 152000)
    T = rng.choice([0.5, 0.7, 1.0])
    size = 4 if dtype == "f32" else 2
    if kind == "stats":
        rows = _logint(rng, 64, 16000)
        rows = min(rows, MAX_BYTES // (V * size))
        return dict(kind=kind, rows=rows, V=V, dtype=dtype, T=T)
    N = _logint(rng, 2, 64)
    tree = kind == "round" and rng.random() < 0.25
    K = rng.choice([24, 48, 64]) if tree else rng.randint(2, 9)
    B = _logint(rng, 1, 64)
    B = max(1, min(B, MAX_BYTES // ((N + 1) * K * V * size)))
    if kind == "round":
        return dict(kind=kind, B=B, N=N, K=K, V=V, dtype=dtype, T=T,
                    mode=rng.choice(["sample", "sample", "greedy"]),
                    loss="length" if tree else rng.choice(["length", "token", "chunk"]), tree=tree)
    if kind == "eval":
        return dict(kind=kind, B=B, N=N, K=K, V=V, dtype=dtype, T=T)
    return dict(kind=kind, B=B, N=N, K=K, V=V, dtype=dtype, T=T, L=rng.choice([4, 8, 10, 16]))


# ---- inputs ------------------------------------------------------------------------------------

def _ld(case):
    return (case["V"] + 7) // 8 * 8


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    return g


def _target(g, B, K, V):
    t = torch.randn((B, K, V), generator=g, device=DEV) * 3.0
    boost = torch.randint(0, V, (B, K, 20), generator=g, device=DEV)
    return t.scatter_add_(2, boost, torch.full(boost.shape, 8.0, device=DEV))


def _logits(case, seed):
    """[N + 1][B][K][ld] logits (row 0 the target), the padding past V zero."""
    B, N, K, V = case["B"], case["N"], case["K"], case["V"]
    g = _generator(seed)
    x = torch.zeros((N + 1, B, K, _ld(case)), dtype=DTYPES[case["dtype"]], device=DEV)
    t = _target(g, B, K, V)
    x[0, :, :, :V] = t
    scales = torch.logspace(math.log10(0.2), math.log10(4.0), N, device=DEV)
    for i in range(N):
        rank = (i + torch.arange(B, device=DEV)) % N
        d = torch.randn((B, K, V), generator=g, device=DEV)
        x[1 + i, :, :, :V] = d.mul_(scales[rank].view(B, 1, 1)).add_(t)
    return x


def _parents(K):
    """Breadth-first draft tree with 3-2-2-2-1-1.. children per level, cut at K nodes."""
    par, level = [-1], [0]
    branching = [3, 2, 2, 2] + [1] * K
    for br in branching:
        nxt = []
        for p in level:
            for _ in range(br):
                if len(par) < K:
                    nxt.append(len(par))
                    par.append(p)
        level = nxt
        if len(par) >= K:
            return par
    return par


def _path_end(case, seed):
    """One random leaf per query."""
    par = _parents(case["K"])
    leaves = sorted(set(range(len(par))) - set(par))
    rng = np.random.default_rng(seed)
    return torch.tensor(rng.choice(leaves, case["B"]), dtype=torch.int32, device=DEV)


def _feedback(case, seed):
    """A stream's state after two rounds, and the feedback of its third."""
    B, N, K = case["B"], case["N"], case["K"]
    g = _generator(seed)
    skill = torch.rand((B, N, 1), generator=g, device=DEV)
    rounds = []
    for _ in range(3):
        a = (skill + 0.3 * torch.randn((B, N, K), generator=g, device=DEV)).clamp_(0.0, 1.0)
        n = torch.randint(1, K + 1, (B,), generator=g, device=DEV, dtype=torch.int32)
        rounds.append((a.contiguous(), n))
    loss = torch.rand((1, B, N), generator=g, device=DEV, dtype=torch.float64)
    eal = 1.0 + K * torch.rand((B, N), generator=g, device=DEV, dtype=torch.float64)
    u = torch.rand((B,), generator=g, device=DEV, dtype=torch.float64)
    return rounds, loss, eal, u


ETA = 0.5


def prepare(case, seed):
    kind = case["kind"]
    if kind == "feedback":
        B, N, K = case["B"], case["N"], case["K"]
        rounds, loss, eal, u = _feedback(case, seed)
        st = hs.DelayedState(B, N, K, DEV)
        for a, n in rounds[:2]:
            hs.delayed_update(st, a, n, ETA)
        return dict(kind=kind, st=st, regret=hs.RegretState(B, N, DEV), gamma=rounds[2][0],
                    count=rounds[2][1], loss=loss, eal=eal, u=u,
                    choice=torch.empty((B,), dtype=torch.int32, device=DEV))
    if kind == "stats":
        g = _generator(seed)
        x = torch.zeros((case["rows"], _ld(case)), dtype=DTYPES[case["dtype"]], device=DEV)
        step = max(1, (1 << 28) // case["V"])
        for r in range(0, case["rows"], step):
            n = min(step, case["rows"] - r)
            x[r:r + n, :case["V"]] = _target(g, n, 1, case["V"])[:, 0]
        return dict(kind=kind, x=x, V=case["V"], T=case["T"])
    if kind == "pruned":
        B, N, K, V, L = case["B"], case["N"], case["K"], case["V"], case["L"]
        g = _generator(seed)
        t = torch.zeros((B, K, _ld(case)), dtype=DTYPES[case["dtype"]], device=DEV)
        t[:, :, :V] = _target(g, B, K, V)
        # each drafter's children: mostly the target's best tokens, some others, some pruned
        top = t[:, :, :V].float().topk(2 * L, dim=2).indices
        pick = torch.argsort(torch.rand((B, N, K, 2 * L), generator=g, device=DEV), dim=3)[..., :L]
        cand = top[:, None].expand(B, N, K, 2 * L).gather(3, pick)
        other = torch.randint(0, V, cand.shape, generator=g, device=DEV)
        r = torch.rand(cand.shape, generator=g, device=DEV)
        cand = torch.where(r < 0.3, other, cand)
        cand = torch.where(r > 0.8, torch.full_like(cand, -1), cand)
        return dict(kind=kind, t=t, cand=cand.to(torch.int32).contiguous(), V=V, T=case["T"],
                    B=B, K=K)
    x = _logits(case, seed)
    if kind == "round":
        tree = case["tree"]
        rnd = hs.Round(x, V=case["V"], temperature=case["T"],
                       mode=hs.SAMPLE if case["mode"] == "sample" else hs.GREEDY,
                       loss_kind=LOSSES[case["loss"]], eta=ETA,
                       parent=_parents(case["K"]) if tree else None,
                       path_end=_path_end(case, seed) if tree else None)
        return dict(kind=kind, round=rnd)
    dt = hs._dtype_code(x)
    if kind == "eval":
        ws = hs.alloc_workspace(case["B"], case["N"], case["K"], case["V"], dt, DEV)
    else:
        n = hs.topl_workspace_size(case["B"], case["N"], case["K"], case["V"], case["L"], dt)
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    return dict(kind=kind, x=x, ws=ws, V=case["V"], T=case["T"], L=case.get("L"))


# ---- one pass ----------------------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "round":
        r = state["round"]
        r.run()
        out = {"eal": r.eal, "loss": r.loss, "logw": r.state.logw, "w": r.state.w,
               "R": r.state.R, "p": r.state.p, "c": r.state.c}
        if r.mode == hs.SAMPLE:
            out["alpha"] = r.alpha
        else:
            out["agree"] = r.agree
        return out
    if kind == "eval":
        return hs.eval_alpha(state["x"], V=state["V"], temperature=state["T"], want_agree=True,
                             want_argmax=True, workspace=state["ws"])
    if kind == "topl":
        return hs.eval_topl(state["x"], L=state["L"], V=state["V"], temperature=state["T"],
                            want_hit=True, want_children=True, workspace=state["ws"])
    if kind == "pruned":
        t = state["t"]
        B, K, ld = t.shape
        _, lse, _ = hs.softmax_stats(t.view(B * K, ld), V=state["V"], temperature=state["T"])
        lse = lse.view(B, K)
        g = hs.candidate_mass(t, lse, state["cand"], V=state["V"], temperature=state["T"])
        return {"lse": lse, "gamma": g}
    if kind == "stats":
        mx, lse, am = hs.softmax_stats(state["x"], V=state["V"], temperature=state["T"])
        return {"max": mx, "lse": lse, "argmax": am}
    st, rg = state["st"], state["regret"]
    hs.delayed_update(st, state["gamma"], state["count"], ETA)
    hs.play(st.learners.p, hs.PLAY_SAMPLE, state["u"], out=state["choice"])
    rg.update(state["loss"], state["choice"], state["eal"])
    return {"w": st.learners.w, "p": st.learners.p, "R": st.learners.R, "choice": state["choice"],
            "regret": rg.regret, "played": rg.played, "eal_sum": rg.eal_sum}


# ---- what a pass cannot do without -------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "feedback":
        B, N, K = case["B"], case["N"], case["K"]
        # ring and feedback, learner state in and out, losses out
        return {"bytes": B * N * (4 * 3 * K + 8 * (2 * 6 + K)), "flops": B * N * K * (2 * K + 60)}
    size = 4 if case["dtype"] == "f32" else 2
    V = case["V"]
    if kind == "stats":
        # per logit: scale, exp2, sum and the argmax compare
        return {"bytes": case["rows"] * (V * size + 12), "flops": 4 * case["rows"] * V}
    B, N, K = case["B"], case["N"], case["K"]
    if kind == "pruned":
        return {"bytes": B * K * V * size + B * N * K * (case["L"] * (4 + size) + 4),
                "flops": 4 * B * K * V}
    logits = (N + 1) * B * K * V
    if kind == "topl":
        return {"bytes": logits * size + B * N * K * (4 * case["L"] + 5), "flops": 2 * logits}
    if kind == "round" and case["mode"] == "greedy":
        return {"bytes": logits * size + B * N * (K + 72), "flops": logits}
    # per logit: scale, exp2 and sum for the normaliser; scale, min and sum for the mass
    return {"bytes": logits * size + B * N * (4 * K + 72), "flops": 6 * logits}


# ---- what another correct implementation would differ by ---------------------------------------

def tolerance(case):
    """About four times what the path shows against `exact` over the ranges above."""
    kind = case["kind"]
    if kind == "feedback" or (kind == "round" and case["mode"] == "greedy"):
        # fp64 throughout; the scale equation is solved to a few ulp
        return {"rel": 1e-11, "differ": 0.0}
    if kind == "round":
        # fp32 masses (alpha 4e-7); NormalHedge's weights amplify them (p 2.6e-6)
        return {"rel": 1e-5, "differ": 0.0}
    if kind == "pruned":
        return {"rel": 4e-6, "differ": 0.0}  # seen: 8.5e-7
    return {"rel": 2e-6, "differ": 0.0}  # seen: alpha 4.6e-7, gamma 1.3e-7, lse 4e-8


# ---- the same numbers in 64 bits ---------------------------------------------------------------

def _first_argmax(x):
    """Lowest index of each row's maximum."""
    m = x.max(dim=-1, keepdim=True).values
    i = torch.arange(x.shape[-1], device=x.device)
    return torch.where(x == m, i, x.shape[-1]).min(dim=-1).values.to(torch.int32)


def _hedge(logw, loss):
    for f in loss:
        logw = logw - ETA * f
    logw = logw - logw.max(dim=1, keepdim=True).values
    return logw, torch.softmax(logw, dim=1)


def _normalhedge(R, p, loss):
    """The L loss vectors in order; c by bisection on s = 1 / c."""
    N = R.shape[1]
    c = torch.zeros(R.shape[0], dtype=torch.float64, device=R.device)
    for f in loss:
        R = R + (p[:, :, None] * (f[:, :, None] - f[:, None, :])).sum(dim=1)
        r2 = R.clamp(min=0.0) ** 2
        M = r2.max(dim=1).values
        ok = M > 0
        Ms = torch.where(ok, M, torch.ones_like(M))
        lo, hi = 2.0 / Ms, 2.0 * (1.0 + math.log(N)) / Ms
        for _ in range(64):
            s = 0.5 * (lo + hi)
            big = torch.exp(0.5 * r2 * s[:, None]).mean(dim=1) > math.e
            lo, hi = torch.where(big, lo, s), torch.where(big, s, hi)
        u = R.clamp(min=0.0) * torch.exp(0.5 * r2 * s[:, None])
        pn = u / u.sum(dim=1, keepdim=True)
        p = torch.where(ok[:, None], pn, torch.full_like(pn, 1.0 / N))
        c = torch.where(ok, 1.0 / s, torch.zeros_like(s))
    return R, p, c


def _accept(gamma, case, seed):
    """Expected accepted lengths [B][N] and losses [L][B][N] of gamma [B][N][K]."""
    B, N, K = gamma.shape
    if case["tree"]:
        par, ends = _parents(K), _path_end(case, seed).tolist()
        pre = torch.empty_like(gamma)
        for n in range(K):
            pre[:, :, n] = gamma[:, :, n] * (pre[:, :, par[n]] if par[n] >= 0 else 1.0)
        eal = torch.ones((B, N), dtype=torch.float64, device=gamma.device)
        length = torch.zeros((B, 1), dtype=torch.float64, device=gamma.device)
        for b, n in enumerate(ends):
            while n >= 0:
                eal[b] += pre[b, :, n]
                length[b] += 1
                n = par[n]
        return eal, (1.0 - eal / (length + 1.0))[None]
    eal = 1.0 + torch.cumprod(gamma, dim=2).sum(dim=2)
    if case["loss"] == "token":
        return eal, (1.0 - gamma).permute(2, 0, 1)
    if case["loss"] == "chunk":
        return eal, (1.0 - gamma).mean(dim=2)[None]
    return eal, (1.0 - eal / (K + 1.0))[None]


def exact(case, seed):
    kind = case["kind"]
    f8 = torch.float64
    if kind == "feedback":
        B, N, K = case["B"], case["N"], case["K"]
        rounds, loss, eal, u = _feedback(case, seed)
        # every query's tokens in order, and the loss of each of its complete windows (zero past
        # a query's last one: a zero vector changes neither learner)
        tokens = [torch.cat([a[b, :, :int(n[b])] for a, n in rounds], dim=1) for b in range(B)]
        windows = max(max(t.shape[1] for t in tokens) - K + 1, 1)
        f = torch.zeros((windows, B, N), dtype=f8, device=DEV)
        for b, t in enumerate(tokens):
            for s in range(t.shape[1] - K + 1):
                eal_s = 1.0 + torch.cumprod(t[:, s:s + K].to(f8), dim=1).sum(dim=1)
                f[s, b] = 1.0 - eal_s / (K + 1.0)
        zero = torch.zeros((B, N), dtype=f8, device=DEV)
        R, p, _ = _normalhedge(zero, torch.full_like(zero, 1.0 / N), f)
        out = {"w": _hedge(zero, f)[1], "p": p, "R": R}
        cum = torch.cumsum(out["p"], dim=1)
        choice = (cum > (u * cum[:, -1])[:, None]).to(torch.int8).argmax(dim=1)
        played = loss[0].gather(1, choice[:, None])[:, 0]
        out.update(choice=choice.to(torch.int32), played=played,
                   regret=played - loss[0].min(dim=1).values,
                   eal_sum=eal.gather(1, choice[:, None])[:, 0])
        return out
    T, V = case["T"], case["V"]
    if kind == "stats":
        x = prepare(case, seed)["x"]
        mx, lse, am = [], [], []
        for r in range(0, x.shape[0], 256):
            z = x[r:r + 256, :V].to(f8)
            mx.append(z.max(dim=1).values)
            lse.append(torch.logsumexp(z / T, dim=1))
            am.append(_first_argmax(z))
        return {"max": torch.cat(mx), "lse": torch.cat(lse), "argmax": torch.cat(am)}
    if kind == "pruned":
        st = prepare(case, seed)
        lse, gamma = [], []
        for b in range(case["B"]):
            z = st["t"][b, :, :V].to(f8) / T  # [K][V]
            ls = torch.logsumexp(z, dim=1)
            cand = st["cand"][b].long()  # [N][K][L]
            p = torch.exp(z - ls[:, None])[None].expand(cand.shape[0], -1, -1)
            m = p.gather(2, cand.clamp(min=0)) * (cand >= 0)
            lse.append(ls)
            gamma.append(m.sum(dim=2))
        return {"lse": torch.stack(lse), "gamma": torch.stack(gamma)}
    x = _logits(case, seed)
    B, N, K = case["B"], case["N"], case["K"]
    want_mass = kind in ("eval", "topl") or case["mode"] == "sample"
    alpha = torch.zeros((B, N, K), dtype=f8, device=DEV)
    agree = torch.zeros((B, N, K), dtype=torch.uint8, device=DEV)
    am_t = torch.zeros((B, K), dtype=torch.int32, device=DEV)
    am_d = torch.zeros((B, N, K), dtype=torch.int32, device=DEV)
    L = case.get("L", 1)
    hit = torch.zeros((B, N, K), dtype=torch.uint8, device=DEV)
    children = torch.zeros((B, N, K, L), dtype=torch.int32, device=DEV)
    index = torch.arange(V, device=DEV)
    for b in range(B):
        t = x[0, b, :, :V].to(f8)
        p = torch.softmax(t / T, dim=1)
        at = _first_argmax(t)
        am_t[b] = at
        for i in range(N):
            raw = x[1 + i, b, :, :V]
            if kind == "topl":
                # a key whose order is (value, lower index first): the fp32 image as an ordered
                # integer (-0 as +0), then the index
                bits = (raw.float() + 0.0).view(torch.int32).long()
                key = torch.where(bits < 0, -(bits & 0x7FFFFFFF), bits) * (1 << 20) - index
                ch = (-(key.topk(L, dim=1).values)) & ((1 << 20) - 1)
                children[b, i] = ch.to(torch.int32)
                hit[b, i] = (ch == at[:, None]).any(dim=1)
                alpha[b, i] = p.gather(1, ch).sum(dim=1)
                continue
            d = raw.to(f8)
            if want_mass:
                alpha[b, i] = torch.minimum(p, torch.softmax(d / T, dim=1)).sum(dim=1)
            if kind == "eval" or case["mode"] == "greedy":
                ad = _first_argmax(d)
                am_d[b, i] = ad
                agree[b, i] = ad == at
    if kind == "eval":
        return {"alpha": alpha, "agree": agree, "argmax_t": am_t, "argmax_d": am_d}
    if kind == "topl":
        return {"gamma": alpha, "hit": hit, "children": children}
    greedy = case["mode"] == "greedy"
    eal, loss = _accept(agree.to(f8) if greedy else alpha, case, seed)
    zero = torch.zeros((B, N), dtype=f8, device=DEV)
    logw, w = _hedge(zero, loss)
    R, p, c = _normalhedge(zero, torch.full_like(zero, 1.0 / N), loss)
    out = {"eal": eal, "loss": loss, "logw": logw, "w": w, "R": R, "p": p, "c": c}
    out["agree" if greedy else "alpha"] = agree if greedy else alpha
    return out
