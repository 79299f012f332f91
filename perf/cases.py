"""The work this library does for its users, as measurable cases.

A case is one call, or the few calls a model's layer makes together, through the
package's public entry points: the whole vector-sparse attention layer (lists,
block order, attention over the gathered keys), a selection whose lists are the
result, an attention over lists that an earlier step selected, a packed batch of
sequences, and the selection that allocates nothing.  Sizes run from the 1k-token
plumbing layer to the 131k-token prefill and the 119k-token video DiT layer.

Inputs are seeded N(0, 1) tensors with planted key columns (the vertical vectors
of real video attention) in the proportions of paper_2603_29494_amd.synth; masks,
head counts and selection parameters are those of that module, of the tests and
of the benchmark, or generic.
"""
import math

import torch

import paper_2603_29494_amd as va
from paper_2603_29494_amd._lib import select_noalloc

DEV = "cuda"

# What each family of inputs plants (synth's workloads 4, 2 / 5 and 3):
#   frames   K: an offset per 1 / 21 of the sequence, 4% columns; Q without a shared direction
#   columns  planted columns along a direction the queries share, chunk offsets on Q and K
#   window   planted columns and a local window of 256 tokens


def listed():
    return [
        # The smallest layer: two heads of 1024 tokens (launches and latency).
        dict(name="layer_1k", kind="layer", B=1, Hq=2, Hkv=2, N=1024, D=64, P=64, causal=False,
             mode="topk", param=0.125, gen="columns", frac=0.03, mu=4.0, keep=0.125),
        # A short prompt in a server that allocates nothing per call: grouped heads, a ragged
        # length, lists by softmax mass.
        dict(name="noalloc_2k", kind="noalloc", B=1, Hq=16, Hkv=4, N=2000, D=128, P=64, causal=True,
             mode="topp", param=0.9, gen="columns", frac=0.04, mu=5.0, keep=0.4),
        # A batch of medium sequences with 64-wide heads (an encoder's layer).
        dict(name="layer_batch_4k", kind="layer", B=4, Hq=12, Hkv=12, N=4096, D=64, P=64,
             causal=False, mode="topk", param=0.2, gen="frames", frac=0.04, mu=2.0, keep=0.2),
        # Prompts of different lengths packed into one prefill.
        dict(name="varlen_28k", kind="varlen", lens="8192,517,3000,12345,64,4111", B=1, Hq=28,
             Hkv=4, N=28229, D=128, P=64, causal=True, mode="topk", param=0.1, gen="columns",
             frac=0.03, mu=4.0, keep=0.1),
        # The paper's own filter (within alpha of the row maximum) at its 17k-token video prompts.
        dict(name="layer_mins_17k", kind="layer", B=1, Hq=32, Hkv=8, N=17000, D=128, P=64,
             causal=True, mode="mins", param=0.3, gen="frames", frac=0.04, mu=2.0, keep=0.2),
        # Algorithm 1's cross-tile filter at the paper's 26k-token prompts; the lists are kept.
        dict(name="select_tiled_26k", kind="select", B=1, Hq=28, Hkv=4, N=26000, D=128, P=64,
             causal=True, mode="mins_tiled", param=0.25, gen="frames", frac=0.04, mu=2.0, keep=0.4),
        # Attention over lists of an earlier denoising step, with the log-sum-exp of every row.
        dict(name="attention_24k", kind="attention", B=1, Hq=24, Hkv=24, N=24001, D=128, P=64,
             causal=False, mode="given", param=0.2, gen="frames", frac=0.04, mu=2.0, keep=0.2),
        # Causal prefill of a vision-language model, 32k tokens, a tenth of the keys.
        dict(name="layer_vlm_32k", kind="layer", B=1, Hq=28, Hkv=4, N=32768, D=128, P=64,
             causal=True, mode="topk", param=0.1, gen="columns", frac=0.03, mu=4.0, keep=0.1),
        # One GPU's share of the 75k-token video DiT layer when eight GPUs split its heads.
        dict(name="layer_dit_75k_shard", kind="layer", B=1, Hq=5, Hkv=5, N=75600, D=128, P=64,
             causal=False, mode="topk", param=0.15, gen="frames", frac=0.04, mu=2.0, keep=0.15),
        # The benchmark: the whole 75k-token video DiT layer.
        dict(name="layer_dit_75k", kind="layer", B=1, Hq=40, Hkv=40, N=75600, D=128, P=64,
             causal=False, mode="topk", param=0.15, gen="frames", frac=0.04, mu=2.0, keep=0.15),
        # Long causal prefill by softmax mass: lists from 2% to most of the keys.
        dict(name="layer_vlm_131k", kind="layer", B=1, Hq=28, Hkv=4, N=131072, D=128, P=64,
             causal=True, mode="topp", param=0.95, gen="window", frac=0.02, mu=8.0, keep=0.22),
        # The 119k-token video DiT layer by softmax mass, 128-row blocks.
        dict(name="layer_dit_119k", kind="layer", B=1, Hq=24, Hkv=24, N=118800, D=128, P=128,
             causal=False, mode="topp", param=0.9, gen="columns", frac=0.045, mu=4.745, keep=0.4),
    ]


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["noalloc", "varlen", "select", "attention"])
    Hkv = rng.choice([1, 2, 3, 4, 5, 8, 10, 12, 24])
    grp = rng.choice([1, 1, 2, 4, 7])
    while Hkv * grp > 40:
        grp = rng.choice([1, 2])
        Hkv = min(Hkv, 20)
    D = rng.choice([64, 128, 128])
    P = rng.choice([32, 48, 64, 64, 64, 128])
    causal = rng.random() < 0.5
    mode = rng.choice(["topk", "topk", "topp", "mins", "mins_tiled"])
    gen = {"topp": "columns", "mins": "frames", "mins_tiled": "frames"}.get(
        mode, rng.choice(["columns", "frames"]))
    hi = {"noalloc": 2500, "varlen": 16000}.get(kind, 118800)
    N = int(round(math.exp(rng.uniform(math.log(600), math.log(hi)))))
    if rng.random() < 0.4:
        N = max(64, N // 64 * 64)
    B = rng.choice([1, 1, 2, 3]) if N < 9000 and kind in ("layer", "select") else 1
    c = dict(kind=kind, B=B, Hq=Hkv * grp, Hkv=Hkv, N=N, D=D, P=P, causal=causal, mode=mode,
             gen=gen, frac=0.04, mu=4.5 if gen == "columns" else 2.0)
    if kind == "varlen":
        n = rng.randint(2, 6)
        lens = [int(round(math.exp(rng.uniform(math.log(40), math.log(hi))))) for _ in range(n)]
        c.update(lens=",".join(str(x) for x in lens), N=sum(lens), mode="topk")
    if kind == "noalloc":
        # its workspace is fixed, at most 64 MiB
        c.update(Hkv=min(c["Hkv"], 4), mode=rng.choice(["topk", "topp"]))
        c["Hq"] = c["Hkv"] * min(grp, 4)
        c.update(gen="columns", mu=4.5)
    if kind == "attention":
        c.update(mode="given")
    param, keep = {"topk": (None, None), "given": (None, None), "topp": (0.9, 0.45),
                   "mins": (0.3, 0.2), "mins_tiled": (0.25, 0.4)}[c["mode"]]
    if param is None:
        param = keep = round(rng.uniform(0.05, 0.3), 3)
    c.update(param=param, keep=keep)
    # no dearer than the largest listed layer, and lists of at most 8 GB
    for h in (c["Hkv"], 12, 8, 5, 4, 2, 1):
        if h <= c["Hkv"]:
            c.update(Hkv=h, Hq=h * (c["Hq"] // c["Hkv"]))
        rows = c["B"] * c["Hq"] * -(-c["N"] // P)
        cap = c["N"] * (c["param"] if c["mode"] in ("topk", "given") else 1.0)
        if work(c)["flops"] < 3e13 and rows * cap * 4 < 8e9:
            break
    return c


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _eligible(N, P, causal):
    Np = -(-N // P)
    return [min(N, (i + 1) * P) if causal else N for i in range(Np)]


def work(case):
    """Bytes: Q, K and V read and O written once (or the lists, where they are the result);
    operations: the pooled scores and the two products over the kept keys."""
    D, P, B, Hq, Hkv, causal = (case[x] for x in ("D", "P", "B", "Hq", "Hkv", "causal"))
    kind, keep, N = case["kind"], case["keep"], case["N"]
    score = attn = kept = 0.0
    for n in _lens(case) if kind == "varlen" else [N]:
        L = _eligible(n, P, causal)
        score += 2.0 * D * B * Hq * sum(L)
        kept += keep * B * Hq * sum(L)
        attn += 4.0 * D * B * Hq * keep * (sum(L) * P - L[-1] * (len(L) * P - n))
    qk, vo = 2.0 * B * N * D * (Hq + Hkv), 2.0 * B * N * D * (Hq + Hkv)
    if kind == "select":
        return {"bytes": qk + 4.0 * kept, "flops": score}
    if kind == "attention":
        return {"bytes": qk + vo + 4.0 * kept + 4.0 * B * Hq * N, "flops": attn}
    return {"bytes": qk + vo, "flops": score + attn}


def _inputs(case, seed):
    """q, k, v in bf16 on the GPU, one head at a time."""
    B, Hq, Hkv, N, D = (case[x] for x in ("B", "Hq", "Hkv", "N", "D"))
    g = torch.Generator(device=DEV).manual_seed(seed)

    def randn(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)

    q = torch.empty(B, Hq, N, D, dtype=torch.bfloat16, device=DEV)
    k = torch.empty(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
    v = torch.empty(B, Hkv, N, D, dtype=torch.bfloat16, device=DEV)
    gen, grp = case["gen"], Hq // Hkv
    window = None
    if gen == "window":  # random Fourier features of a 256-token window, 2 logits at the diagonal
        w = torch.randn(D, generator=g, device=DEV, dtype=torch.float64) / 256.0
        ph = torch.rand(D, generator=g, device=DEV, dtype=torch.float64) * (2.0 * math.pi)
        t = torch.arange(N, device=DEV, dtype=torch.float64)[:, None]
        window = (math.sqrt(2.0 / D) * torch.cos(t * w + ph)).float()
        window *= math.sqrt(2.0 * math.sqrt(D))
    step = max(1, N // 21) if gen == "frames" else 1024
    for b in range(B):
        for h in range(Hkv):
            u = randn(D)
            u /= u.norm()
            planted = torch.rand(N, generator=g, device=DEV) < case["frac"]
            kk = randn(N, D)
            off = 0.0
            if gen != "window":
                sigma = 0.5 if gen == "frames" else D ** -0.25
                off = (randn(-(-N // step), D) * sigma).repeat_interleave(step, 0)[:N]
                kk += off
            else:
                kk += window
            kk += planted[:, None] * (case["mu"] * math.sqrt(D)) * u
            k[b, h] = kk
            v[b, h] = randn(N, D)
            for j in range(grp):
                qq = randn(N, D)
                if gen == "columns":
                    qq += u + off
                elif gen == "window":
                    qq += u + window
                q[b, h * grp + j] = qq
    return q, k, v, g


def _given_lists(case, seed, g):
    """Lists an earlier step selected: random ascending keys, the same number for every block,
    a share of them common to the blocks of a head (planted columns)."""
    B, Hq, N, P = (case[x] for x in ("B", "Hq", "N", "P"))
    Np = -(-N // P)
    cap = max(1, int(case["param"] * N))
    idx = torch.empty(B, Hq, Np, cap, dtype=torch.int32, device=DEV)
    counts = torch.full((B, Hq, Np), cap, dtype=torch.int32, device=DEV)
    for b in range(B):
        for h in range(Hq):
            common = (torch.rand(N, generator=g, device=DEV) < case["frac"]).float()
            x = torch.rand(Np, N, generator=g, device=DEV) + common
            idx[b, h] = x.topk(cap, dim=1).indices.sort(dim=1).values.int()
    return idx, counts


def prepare(case, seed):
    q, k, v, g = _inputs(case, seed)
    B, Hq, N, P, causal = (case[x] for x in ("B", "Hq", "N", "P", "causal"))
    Np = -(-N // P)
    s = dict(case=case, q=q, k=k, v=v)
    if case["kind"] == "attention":
        s["idx"], s["counts"] = _given_lists(case, seed, g)
        return s
    if case["kind"] == "varlen":
        cu = [0]
        for n in _lens(case):
            cu.append(cu[-1] + n)
        s["cu"] = cu
        s["cap"] = max(va.max_count(n, P, causal, case["mode"], case["param"]) for n in _lens(case))
        return s
    cap = va.max_count(N, P, causal, case["mode"], case["param"])
    s["cap"] = cap
    s["idx"] = torch.empty(B, Hq, Np, cap, dtype=torch.int32, device=DEV)
    s["counts"] = torch.empty(B, Hq, Np, dtype=torch.int32, device=DEV)
    if case["kind"] != "noalloc":
        s["ws"] = torch.empty(va.workspace_bytes(q, k, P, causal, case["mode"], cap),
                              dtype=torch.uint8, device=DEV)
    if case["kind"] != "select":
        s["order"] = torch.empty(B, Hq, Np, dtype=torch.int32, device=DEV)
        s["o"] = torch.empty_like(q)
    return s


def run(s):
    c = s["case"]
    q, k, v, P, causal = s["q"], s["k"], s.get("v"), c["P"], c["causal"]
    if c["kind"] == "attention":
        o, lse = va.sparse_attn(q, k, v, s["idx"], s["counts"], P, causal, return_lse=True)
        return {"o": o, "lse": lse}
    if c["kind"] == "varlen":
        idx, counts = va.select_varlen(q, k, s["cu"], P, c["mode"], c["param"], causal)
        o = va.sparse_attn_varlen(q, k, v, s["cu"], idx, counts, s["cap"], P, causal)
        return {"o": o, "counts": counts}
    if c["kind"] == "select":
        idx, counts = va.select(q, k, P, c["mode"], c["param"], causal, cap=s["cap"], idx=s["idx"],
                                counts=s["counts"], workspace=s["ws"])
        return {"idx": idx, "counts": counts}
    if c["kind"] == "noalloc":
        select_noalloc(q, k, P, c["mode"], c["param"], causal, s["cap"], s["idx"], s["counts"])
    else:
        va.select(q, k, P, c["mode"], c["param"], causal, cap=s["cap"], idx=s["idx"],
                  counts=s["counts"], workspace=s["ws"], unpadded=True)
    va.attn_order(s["idx"], s["counts"], c["N"], P, out=s["order"])
    va.sparse_attn(q, k, v, s["idx"], s["counts"], P, causal, out=s["o"], order=s["order"])
    return {"o": s["o"], "counts": s["counts"]}


def tolerance(case):
    """Outputs are bf16, and their softmax weights are rounded to bf16 before the product with V;
    scores are fp32, so keys within an ulp or so of a cut can go either way, which changes the
    outputs of those blocks, the counts (mass and threshold modes) and, in a list, the places of
    the keys after them."""
    return {"rel": 0.012, "max": 0.2, "differ": 0.01}


def _lists64(q, k, P, causal, mode, param):
    """Boolean kept-key map [Np, N] of one head in 64 bits."""
    N, D = q.shape
    Np = -(-N // P)
    pad = torch.zeros(Np * P, D, dtype=torch.float64, device=q.device)
    pad[:N] = q.double()
    n = torch.full((Np, 1), float(P), dtype=torch.float64, device=q.device)
    n[-1] = N - (Np - 1) * P
    qp = (pad.view(Np, P, D).sum(1) / n).to(torch.bfloat16).double()
    s = qp @ k.double().t() / math.sqrt(D)
    L = torch.tensor(_eligible(N, P, causal), device=q.device)
    s.masked_fill_(torch.arange(N, device=q.device)[None, :] >= L[:, None], -math.inf)
    if mode == "mins":
        return s >= s.max(1, keepdim=True).values - param
    if mode == "mins_tiled":  # tiles of 16 keys in groups of 16
        G = -(-N // 256)
        t = torch.full((Np, G * 256), -math.inf, dtype=torch.float64, device=q.device)
        t[:, :N] = s
        m = t.view(Np, G, 16, 16).max(3).values.cummax(2).values
        thr = (m - param).repeat_interleave(16, 2).reshape(Np, -1)[:, :N]
        return (s >= thr) & (s > -math.inf)
    v, at = s.sort(dim=1, descending=True, stable=True)
    if mode == "topk":
        cnt = torch.ceil(param * L.double() - 1e-9).clamp(min=1).minimum(L.double())
    else:
        p = torch.softmax(v, 1)
        cnt = ((p.cumsum(1) < param).sum(1) + 1).double().minimum(L.double())
    first = torch.arange(N, device=q.device)[None, :] < cnt[:, None]
    return torch.zeros_like(first).scatter_(1, at, first)


def _attend64(q, k, v, kept, P, causal, o, lse):
    """Attention over the kept keys of one head in 64 bits, a group of blocks of like list
    length at a time."""
    N, D = q.shape
    cnt = kept.sum(1)
    kd, vd = k.double(), v.double()
    order = cnt.argsort().tolist()
    width = cnt.tolist()
    at = 0
    while at < len(order):
        m = max(1, int(2 ** 27 // max(1, D * width[order[min(at + 15, len(order) - 1)]])))
        blocks = order[at:at + min(m, 256)]
        at += len(blocks)
        nb, W = len(blocks), max(1, width[blocks[-1]])
        bt = torch.tensor(blocks, device=q.device)
        rank = kept[bt].int().cumsum(1) - 1
        r, c = kept[bt].nonzero(as_tuple=True)
        ids = torch.full((nb, W), N, device=q.device)
        ids[r, rank[r, c].long()] = c
        rows = bt[:, None] * P + torch.arange(P, device=q.device)
        live = ids < N
        safe = ids.clamp(max=N - 1)
        kg = kd[safe.view(-1)].view(nb, W, D).transpose(1, 2).contiguous()
        s = torch.bmm(q[rows.clamp(max=N - 1).view(-1)].double().view(nb, P, D), kg) / math.sqrt(D)
        del kg
        mask = live[:, None, :].expand(nb, P, W)
        if causal:
            mask = mask & (ids[:, None, :] <= rows[:, :, None])
        s.masked_fill_(~mask, -math.inf)
        l = torch.logsumexp(s, 2)
        w = torch.exp(s - torch.where(l == -math.inf, torch.zeros_like(l), l)[:, :, None])
        del s
        out = torch.bmm(w, vd[safe.view(-1)].view(nb, W, D))
        ok = (rows < N).view(-1)
        o[rows.view(-1)[ok]] = out.reshape(-1, D)[ok]
        lse[rows.view(-1)[ok]] = l.reshape(-1)[ok]


def exact(case, seed):
    if work(case)["flops"] > 2.5e13 or case["kind"] == "select":
        return None
    q, k, v, g = _inputs(case, seed)
    B, Hq, Hkv, N, P, causal = (case[x] for x in ("B", "Hq", "Hkv", "N", "P", "causal"))
    o = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.empty(B, Hq, N, dtype=torch.float64, device=DEV)
    given = _given_lists(case, seed, g)[0] if case["kind"] == "attention" else None
    spans, at = [], 0
    for n in _lens(case) if case["kind"] == "varlen" else [N]:
        spans.append((at, at + n))
        at += n
    for b in range(B):
        for h in range(Hq):
            kk, vv = k[b, h // (Hq // Hkv)], v[b, h // (Hq // Hkv)]
            for a, z in spans:
                if given is not None:
                    kept = torch.zeros(given.shape[2], N, dtype=torch.bool, device=DEV)
                    kept.scatter_(1, given[b, h].long(), True)
                else:
                    kept = _lists64(q[b, h, a:z], kk[a:z], P, causal, case["mode"], case["param"])
                _attend64(q[b, h, a:z], kk[a:z], vv[a:z], kept, P, causal, o[b, h, a:z],
                          lse[b, h, a:z])
    return {"o": o, "lse": lse} if given is not None else {"o": o, "counts": None}
