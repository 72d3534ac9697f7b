"""The work that users of this library have it do, as cases that can be timed and compared.

Four kinds of call, each through the binding that programs use (``paper_2511_12934_amd.binding``):

* ``score``: the real-time phase of a pre-ranking request -- gather, target attention, cross features, MLP head and the
  cut to the k best (``aif_score_topk``; a candidate list cut into 1,000-item mini-batches goes through
  ``aif_score_batch`` and one ``aif_topk``),
* ``user``: the user-side network that runs beside retrieval (``aif_user_precompute``),
* ``lsh``: long-sequence behaviour modelling on signatures (``aif_lsh_batch``),
* ``update``: the nearline refresh of table rows (``aif_update_rows``), and ``topk``: the selection alone (``aif_topk``).

Shapes are those of the library's own configurations; inputs are drawn on the device with the configurations'
distributions: values N(0, 0.1), Xavier-uniform weights, candidate ids uniform or Zipf(1.1) and distinct within a request.
"""
import functools
import math

import torch

from paper_2511_12934_amd import binding as B

DEV = "cuda:0"
NONE, HADAMARD, SEGDOT, BEA = 0, 1, 2, 3

# model shapes of the scoring path, by the name the library's workloads give them
MODELS = {
    # one small request; also the shape that stands for "widths without kernels of their own" in bf16
    "C1": dict(d_item=64, d_user=64, d_attn=32, heads=1, wq=True, cross=HADAMARD, n_cross=0, d_cv=0,
               mlp=(224, 128, 64, 1), k=100, ids="uniform"),
    "C2": dict(d_item=64, d_user=64, d_attn=64, heads=1, wq=False, cross=HADAMARD, n_cross=0, d_cv=0,
               mlp=(256, 256, 128, 1), k=200, ids="zipf"),
    "C3": dict(d_item=64, d_user=64, d_attn=64, heads=1, wq=False, cross=HADAMARD, n_cross=0, d_cv=0,
               mlp=(256, 512, 256, 1), k=100, ids="zipf"),
    "C4": dict(d_item=128, d_user=128, d_attn=128, heads=4, wq=False, cross=HADAMARD, n_cross=0, d_cv=0,
               mlp=(512, 256, 1), k=100, ids="uniform"),
    "C5": dict(d_item=256, d_user=576, d_attn=128, heads=8, wq=True, cross=SEGDOT, n_cross=16, d_cv=64,
               mlp=(1024, 1024, 512, 256, 1), k=150, ids="zipf"),
    "B3": dict(d_item=64, d_user=64, d_attn=64, heads=1, wq=False, cross=BEA, n_cross=16, d_cv=64,
               mlp=(256, 512, 256, 1), k=100, ids="zipf"),
}


def listed():
    return [
        # the smallest request there is: one mini-batch of 1,000 candidates, fp32; latency and launches count
        dict(name="f32 one mini-batch", path="score", model="C1", dtype="f32", users=1, cand=1000, seq=50, items=100_000, ragged=False, slices=False),
        # fp32 models under load: concurrent users whose lists and histories differ in length
        dict(name="f32 16 ragged users", path="score", model="C1", dtype="f32", users=16, cand=10_000, seq=50, items=1_000_000, ragged=True, slices=False),
        # a bf16 model whose head and attention widths are not among the tuned ones
        dict(name="bf16 small model 16 users", path="score", model="C1", dtype="bf16", users=16, cand=10_000, seq=50, items=1_000_000, ragged=False, slices=False),
        # the latency of one whole request over a long history
        dict(name="one request L=1000", path="score", model="C2", dtype="bf16", users=1, cand=10_000, seq=1000, items=1_000_000, ragged=False, slices=False),
        # the batched serving load
        dict(name="64 users", path="score", model="C3", dtype="bf16", users=64, cand=10_000, seq=500, items=10_000_000, ragged=False, slices=False),
        # a table far beyond the caches, uniform ids, short histories, several heads
        dict(name="16 users 12.8 GB table", path="score", model="C4", dtype="bf16", users=16, cand=20_000, seq=200, items=50_000_000, ragged=False, slices=False),
        # the wide model: projected queries, 8 heads, long histories, three wide layers
        dict(name="32 users wide model", path="score", model="C5", dtype="bf16", users=32, cand=10_000, seq=2000, items=10_000_000, ragged=False, slices=False),
        # bridge-embedding cross, odd counts: 37 users with lists and histories of every length
        dict(name="37 ragged users bridges", path="score", model="B3", dtype="bf16", users=37, cand=9_973, seq=499, items=10_000_000, ragged=True, slices=False),
        # the asynchronous user side of the batched load
        dict(name="user network 64 users", path="user", dtype="bf16", users=64, seq=500, raw=128, d=64),
        # signature modelling of a 10^4-item history for 64 users
        dict(name="signatures 10^4 history", path="lsh", dtype="bf16", users=64, cand=10_000, seq=10_000, items=10_000_000, bits=64, d=64, tiers=8, ragged=False),
        # ... and of a 10^5-item history with wider signatures for 8
        dict(name="signatures 10^5 history", path="lsh", dtype="bf16", users=8, cand=10_000, seq=100_000, items=10_000_000, bits=128, d=128, tiers=8, ragged=False),
        # the nearline refresh of a tenth of the table
        dict(name="update 10^6 rows", path="update", dtype="bf16", items=10_000_000, rows=1_000_000, d=64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the listed ones' ranges: fewer users, shorter lists and histories, ragged or not, cut or whole."""
    what = rng.choice(["score"] * 10 + ["user"] * 2 + ["lsh"] * 3 + ["update", "topk"])
    ragged = rng.random() < 0.5
    if what == "score":
        # (model, type, most users, most candidates, longest history, table rows)
        model, dtype, users, cand, seq, items = rng.choice([
            ("C1", "f32", 16, 10_000, 200, 1_000_000), ("C1", "f32", 1, 10_000, 200, 100_000), ("C1", "bf16", 16, 10_000, 200, 1_000_000),
            ("C3", "f32", 2, 4_000, 200, 1_000_000), ("C2", "bf16", 4, 10_000, 1500, 1_000_000), ("C2", "bf16", 1, 10_000, 1000, 1_000_000),
            ("C3", "bf16", 64, 10_000, 500, 10_000_000), ("C4", "bf16", 16, 20_000, 200, 50_000_000),
            ("C5", "bf16", 32, 10_000, 2000, 10_000_000), ("B3", "bf16", 64, 10_000, 500, 10_000_000)])
        n = _log(rng, 50, cand)
        return dict(path="score", model=model, dtype=dtype, users=_log(rng, 1, users), cand=n, seq=_log(rng, 8, seq),
                    items=_log(rng, 40_000, items), ragged=ragged, slices=n > 1000 and rng.random() < 0.25)
    if what == "user":
        raw, d = rng.choice([(128, 64), (64, 64), (48, 32)])
        dtype = rng.choice(["bf16", "bf16", "f32"])
        return dict(path="user", dtype=dtype, users=_log(rng, 1, 64 if dtype == "bf16" else 8), seq=_log(rng, 8, 500), raw=raw, d=d)
    if what == "lsh":
        bits, d, users, seq = rng.choice([(64, 64, 64, 10_000), (128, 128, 8, 100_000), (64, 64, 1, 10_000)])
        return dict(path="lsh", dtype=rng.choice(["bf16", "bf16", "f32"]), users=_log(rng, 1, users), cand=_log(rng, 100, 10_000),
                    seq=_log(rng, 500, seq), items=_log(rng, 100_000, 10_000_000), bits=bits, d=d, tiers=8, ragged=ragged)
    if what == "update":
        items = _log(rng, 100_000, 10_000_000)
        return dict(path="update", dtype=rng.choice(["bf16", "f32"]), items=items, rows=_log(rng, 500, items // 10), d=rng.choice([64, 128]))
    return dict(path="topk", lists=_log(rng, 1, 64), n=_log(rng, 100, 20_000), k=rng.choice([10, 100, 200]))


# ---------------------------------------------------------------------------
# sizes of one case
# ---------------------------------------------------------------------------
def _spread(n, r, lowest):
    """Length of user r's list in a ragged batch: between a quarter of n and n, fixed by r alone."""
    return max(lowest, n - int(0.75 * n * ((r * 0.6180339887) % 1.0)))


def _sizes(c):
    """Per user: candidates, history length."""
    if not c["ragged"]:
        return [c["cand"]] * c["users"], [c["seq"]] * c["users"]
    return ([_spread(c["cand"], r, 1) for r in range(c["users"])],
            [_spread(c["seq"], r + 7, 1) for r in range(c["users"])])


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (int(seed) + 1))
    return g


def _normal(g, shape, dt, sigma=0.1):
    out = torch.empty(shape, dtype=dt, device=DEV)
    flat = out.view(-1)
    for lo in range(0, flat.numel(), 1 << 30):
        flat[lo:lo + (1 << 30)].normal_(0.0, sigma, generator=g)
    return out


def _xavier(g, n_out, n_in, dt):
    lim = math.sqrt(6.0 / (n_in + n_out))
    return torch.empty((n_out, n_in), device=DEV).uniform_(-lim, lim, generator=g).to(dt)


@functools.lru_cache(maxsize=4)
def _zipf_cdf(n):
    p = torch.arange(1, n + 1, dtype=torch.float64, device=DEV).pow_(-1.1).cumsum_(0)
    return p / p[-1]


def _ids(g, how, n_items, users, n):
    """[users, n] row numbers, distinct within a user: drawn until n different ones have come up."""
    m = n + n // 4 + 64 if how == "uniform" else 6 * n + 64
    while True:
        if how == "uniform":
            d = torch.randint(0, n_items, (users, m), device=DEV, generator=g)
        else:
            u = torch.rand((users, m), device=DEV, dtype=torch.float64, generator=g)
            d = torch.searchsorted(_zipf_cdf(n_items), u).clamp_(max=n_items - 1)
        v, at = torch.sort(d, dim=1, stable=True)
        first = torch.ones_like(v, dtype=torch.bool)
        first[:, 1:] = v[:, 1:] != v[:, :-1]
        keep = torch.zeros_like(first).scatter_(1, at, first)
        place = keep.cumsum(1)
        if int(place[:, -1].min()) >= n:
            d = d[keep & (place <= n)].view(users, n)
            step = 2_654_435_761                       # hot rows lie scattered over the table
            while math.gcd(step, n_items) != 1:
                step += 2
            return ((d * step + 12345) % n_items).to(torch.int32)
        m *= 2


# ---------------------------------------------------------------------------
# the scoring path
# ---------------------------------------------------------------------------
def _score_inputs(c, seed):
    M, dt, g = MODELS[c["model"]], _dt(c), _gen(seed)
    ns, ls = _sizes(c)
    table = _normal(g, (c["items"], M["d_item"]), dt)
    if M["cross"] == BEA:                               # a row ends with its bridge weights: non-negative, summing to one
        for lo in range(0, c["items"], 1 << 22):
            w = torch.empty((min(1 << 22, c["items"] - lo), M["n_cross"]), device=DEV).exponential_(generator=g)
            table[lo:lo + (1 << 22), M["d_item"] - M["n_cross"]:] = (w / w.sum(1, keepdim=True)).to(dt)
    ids = _ids(g, M["ids"], c["items"], c["users"], max(ns))
    ws = [_xavier(g, M["mlp"][i + 1], M["mlp"][i], dt) for i in range(len(M["mlp"]) - 1)]
    bs = [_normal(g, (n,), dt, 0.05) for n in M["mlp"][1:]]
    wq = _xavier(g, M["d_attn"], M["d_item"], dt) if M["wq"] else None
    users = [dict(u=_normal(g, (M["d_user"],), dt), k=_normal(g, (ls[r], M["d_attn"]), dt), v=_normal(g, (ls[r], M["d_attn"]), dt),
                  x=_normal(g, (M["n_cross"], M["d_cv"]), dt) if M["n_cross"] else None,
                  ids=ids[r, :ns[r]].contiguous()) for r in range(c["users"])]
    return table, ws, bs, wq, users


def _prepare_score(c, seed):
    M = MODELS[c["model"]]
    table, ws, bs, wq, users = _score_inputs(c, seed)
    ns, ls = _sizes(c)
    total = sum(ns)
    logits, scores = torch.zeros(total, device=DEV), torch.zeros(total, device=DEV)
    idx = torch.zeros((c["users"], M["k"]), dtype=torch.int32, device=DEV)
    val = torch.zeros((c["users"], M["k"]), device=DEV)
    reqs, whole, at = [], [], 0
    for u, n in zip(users, ns):
        z, y = logits[at:at + n], scores[at:at + n]
        at += n
        whole.append(z)
        step = 1000 if c["slices"] else n
        for lo in range(0, n, step):
            reqs.append(B.Request(u["u"], u["k"], u["v"], u["ids"][lo:lo + step], z[lo:lo + step], y[lo:lo + step], u["x"]))
    ctx = B.Context(dtype=B.AIF_F32 if c["dtype"] == "f32" else B.AIF_BF16, table=table, d_user=M["d_user"], d_attn=M["d_attn"],
                    n_heads=M["heads"], max_seq_len=max(ls), layer_dims=list(M["mlp"]), weights=ws, biases=bs, w_q=wq,
                    cross_mode=M["cross"], n_cross=M["n_cross"], d_cross_vec=M["d_cv"], max_candidates=max(q.n_cand for q in reqs),
                    max_users=len(reqs))
    return dict(run=_run_score, ctx=ctx, reqs=reqs, packed=B.pack_requests(reqs), whole=whole, slices=c["slices"], k=M["k"],
                idx=idx, val=val, logits=logits, scores=scores, f32=c["dtype"] == "f32", keep=(table, ws, bs, wq, users))


def _run_score(s):
    if s["slices"]:
        s["ctx"].aif_score_batch(s["reqs"], packed=s["packed"])
        s["ctx"].aif_topk(s["whole"], s["k"], s["idx"], s["val"])
    else:
        s["ctx"].aif_score_topk(s["reqs"], s["k"], s["idx"], s["val"], packed=s["packed"])
    out = {"logits": s["logits"], "scores": s["scores"], "best": s["val"]}
    if s["f32"]:        # bf16 logits lie so close that any rounding swaps neighbours: positions are compared in fp32 and for topk alone
        out["positions"] = s["idx"]
    return out


def _exact_score(c, seed):
    M = MODELS[c["model"]]
    table, ws, bs, wq, users = _score_inputs(c, seed)
    ws, bs = [w.double() for w in ws], [b.double() for b in bs]
    H, dh, S = M["heads"], M["d_attn"] // M["heads"], M["d_item"] // M["d_cv"] if M["d_cv"] else 0
    logits, best, pos = [], [], []
    for u in users:
        z_all = []
        K, V, uv = u["k"].double(), u["v"].double(), u["u"].double()
        for lo in range(0, u["ids"].numel(), 10_000):
            e = table[u["ids"][lo:lo + 10_000].long()].double()
            q = e @ wq.double().t().contiguous() if wq is not None else e[:, :M["d_attn"]]
            a = []
            for h in range(H):
                cols = slice(h * dh, (h + 1) * dh)
                p = torch.softmax(q[:, cols].contiguous() @ K[:, cols].t().contiguous() / math.sqrt(dh), dim=1)
                a.append(p @ V[:, cols].contiguous())
            if M["cross"] == HADAMARD:
                x = e * uv
            elif M["cross"] == SEGDOT:
                cv = u["x"].double().t().contiguous()
                x = torch.stack([e[:, s * M["d_cv"]:(s + 1) * M["d_cv"]].contiguous() @ cv for s in range(S)], dim=2).reshape(e.shape[0], -1)
            else:
                x = e[:, M["d_item"] - M["n_cross"]:].contiguous() @ u["x"].double()
            y = torch.cat([uv.expand(e.shape[0], -1), e] + a + [x], dim=1)
            for l, (w, b) in enumerate(zip(ws, bs)):
                y = y @ w.t().contiguous() + b
                if l + 1 < len(ws):
                    y = y.relu()
            z_all.append(y[:, 0])
        z = torch.cat(z_all)
        logits.append(z)
        v, at = torch.sort(z, descending=True, stable=True)
        k, n = M["k"], z.numel()
        best.append(torch.cat([v[:k], v.new_full((max(0, k - n),), -math.inf)]))
        pos.append(torch.cat([at[:k], at.new_full((max(0, k - n),), -1)]))
    logits = torch.cat(logits)
    out = {"logits": logits, "scores": torch.sigmoid(logits), "best": torch.stack(best)}
    if c["dtype"] == "f32":
        out["positions"] = torch.stack(pos).to(torch.int32)
    return out


def _work_score(c):
    M, esz = MODELS[c["model"]], 4 if c["dtype"] == "f32" else 2
    ns, ls = _sizes(c)
    n = sum(ns)
    # what depends on the user alone, and what is bilinear in user and item, is done once per user: layer 1 contracts
    # over [item | attention] per candidate
    mlp = M["mlp"]
    head = (M["d_item"] + M["d_attn"]) * mlp[1] + sum(a * b for a, b in zip(mlp[1:-1], mlp[2:]))
    flops = n * 2 * (head + (M["d_item"] * M["d_attn"] if M["wq"] else 0)) + sum(4 * a * b * M["d_attn"] for a, b in zip(ns, ls))
    weights = sum(a * b for a, b in zip(mlp[:-1], mlp[1:])) + (M["d_item"] * M["d_attn"] if M["wq"] else 0)
    moved = n * (4 + M["d_item"] * esz + 4 + 4) + esz * (weights + sum(2 * l * M["d_attn"] + M["d_user"] + M["n_cross"] * M["d_cv"] for l in ls))
    return {"bytes": moved + 8 * M["k"] * c["users"], "flops": flops}


# ---------------------------------------------------------------------------
# the user-side network
# ---------------------------------------------------------------------------
def _user_inputs(c, seed):
    g, dt, d, raw = _gen(seed), _dt(c), c["d"], c["raw"]
    w = dict(p=_xavier(g, d, raw, dt), s=_xavier(g, d, raw, dt), f=_xavier(g, d, d, dt), b=_normal(g, (d,), dt, 0.05))
    lens = [_spread(c["seq"], r, 1) if r % 2 else c["seq"] for r in range(c["users"])]      # histories of every length
    return w, lens, [(_normal(g, (raw,), dt), _normal(g, (l, raw), dt)) for l in lens]


def _prepare_user(c, seed):
    w, lens, users = _user_inputs(c, seed)
    vec = torch.zeros((c["users"], 2 * c["d"]), dtype=_dt(c), device=DEV)
    seq = torch.zeros((sum(lens), c["d"]), dtype=_dt(c), device=DEV)
    reqs, at = [], 0
    for r, ((p, s), l) in enumerate(zip(users, lens)):
        reqs.append(B.UserRequest(p, s, vec[r], seq[at:at + l]))
        at += l
    ctx = B.UserContext(dtype=B.AIF_F32 if c["dtype"] == "f32" else B.AIF_BF16, d_raw=c["raw"], d=c["d"], w_profile=w["p"], w_seq=w["s"],
                        w_ffn=w["f"], b_ffn=w["b"], max_seq_len=max(lens), max_users=c["users"])
    return dict(run=_run_user, ctx=ctx, reqs=reqs, packed=B.pack_user_requests(reqs), vec=vec, seq=seq, keep=(w, users))


def _run_user(s):
    s["ctx"].aif_user_precompute(s["reqs"], packed=s["packed"])
    return {"vec": s["vec"], "seq": s["seq"]}


def _exact_user(c, seed):
    w, lens, users = _user_inputs(c, seed)
    w = {k: v.double() for k, v in w.items()}
    vec, seq, root = [], [], math.sqrt(c["d"])
    for p, s in users:
        up, us = w["p"] @ p.double(), s.double() @ w["s"].t().contiguous()
        ust = us.t().contiguous()
        y = (torch.softmax(us @ ust / root, dim=1) @ us) @ w["f"].t().contiguous() + w["b"]
        vec.append(torch.cat([y.relu().mean(0), torch.softmax(up @ ust / root, dim=0) @ us]))
        seq.append(us)
    return {"vec": torch.stack(vec), "seq": torch.cat(seq)}


def _work_user(c):
    esz, d, raw = 4 if c["dtype"] == "f32" else 2, c["d"], c["raw"]
    lens = [_spread(c["seq"], r, 1) if r % 2 else c["seq"] for r in range(c["users"])]
    return {"bytes": sum(esz * ((l + 1) * raw + (l + 2) * d) for l in lens) + esz * (2 * raw * d + d * d),
            "flops": sum(2 * (l + 1) * raw * d + 4 * (l + 1) * l * d + 2 * l * d * d for l in lens)}


# ---------------------------------------------------------------------------
# signature modelling
# ---------------------------------------------------------------------------
def _flip(g, protos, which):
    """Signatures of items of the clusters `which`: the cluster's bits, each flipped with probability 0.15."""
    n, nbytes = which.numel(), protos.shape[1]
    place = 2 ** torch.arange(8, device=DEV, dtype=torch.int32)
    out = torch.empty((n, nbytes), dtype=torch.uint8, device=DEV)
    for lo in range(0, n, 1 << 20):
        m = min(1 << 20, n - lo)
        flips = ((torch.rand((m, nbytes, 8), device=DEV, generator=g) < 0.15).to(torch.int32) * place).sum(2).to(torch.uint8)
        out[lo:lo + m] = protos[which[lo:lo + m]] ^ flips
    return out


def _lsh_inputs(c, seed):
    g = _gen(seed)
    protos = torch.randint(0, 256, (64, c["bits"] // 8), device=DEV, generator=g).to(torch.uint8)
    table = _flip(g, protos, torch.arange(c["items"], device=DEV) % 64)
    ns, ls = _sizes(c)
    ids = _ids(g, "uniform", c["items"], c["users"], max(ns))
    users = []
    for r in range(c["users"]):                       # a user's history comes from eight favoured clusters
        fav = torch.randperm(64, device=DEV, generator=g)[:8]
        sig = _flip(g, protos, fav[torch.randint(0, 8, (ls[r],), device=DEV, generator=g)])
        users.append((sig, _normal(g, (ls[r], c["d"]), _dt(c)), ids[r, :ns[r]].contiguous()))
    return table, users


def _prepare_lsh(c, seed):
    table, users = _lsh_inputs(c, seed)
    ns, ls = _sizes(c)
    din = torch.zeros((sum(ns), c["d"]), device=DEV)
    tier = torch.zeros((sum(ns), c["tiers"]), dtype=torch.int32, device=DEV)
    reqs, at = [], 0
    for (sig, emb, ids), n in zip(users, ns):
        reqs.append(B.LshRequest(sig, emb, ids, din[at:at + n], tier[at:at + n]))
        at += n
    ctx = B.LshContext(sig_table=table, d_out=c["d"], n_tiers=c["tiers"], dtype=B.AIF_F32 if c["dtype"] == "f32" else B.AIF_BF16,
                       max_seq_len=max(ls), max_candidates=max(ns), max_users=c["users"])
    return dict(run=_run_lsh, ctx=ctx, reqs=reqs, packed=B.pack_lsh_requests(reqs), din=din, tier=tier, keep=(table, users))


def _run_lsh(s):
    s["ctx"].aif_lsh_batch(s["reqs"], packed=s["packed"])
    return {"din": s["din"], "tiers": s["tier"]}


def _signs(sig):
    bits = (sig.to(torch.int32).unsqueeze(2) >> torch.arange(8, device=DEV)) & 1
    return (2 * bits.reshape(sig.shape[0], -1) - 1).float()


def _exact_lsh(c, seed):
    table, users = _lsh_inputs(c, seed)
    din, tiers, db, N = [], [], c["bits"], c["tiers"]
    for sig, emb, ids in users:
        hist, emb = _signs(sig).t().contiguous(), emb.double()
        for lo in range(0, ids.numel(), 1000):
            dots = _signs(table[ids[lo:lo + 1000].long()]) @ hist              # whole numbers up to 256: exact in fp32
            same = ((dots + db) / 2).round().to(torch.int32)                  # equal bits
            t = ((same * N) // db).clamp_(max=N - 1).to(torch.uint8)
            tiers.append(torch.stack([(t == i).sum(1) for i in range(N)], dim=1).to(torch.int32))
            din.append((same.double() / db) @ emb)
    return {"din": torch.cat(din), "tiers": torch.cat(tiers)}


def _work_lsh(c):
    esz = 4 if c["dtype"] == "f32" else 2
    ns, ls = _sizes(c)
    n = sum(ns)
    pairs = sum(a * b for a, b in zip(ns, ls))
    return {"bytes": n * (4 + c["bits"] // 8 + 4 * c["d"] + 4 * c["tiers"]) + sum(ls) * (c["bits"] // 8 + esz * c["d"]),
            "flops": 2 * c["bits"] * pairs + 2 * c["bits"] * c["d"] * (n + sum(ls))}


# ---------------------------------------------------------------------------
# table rows, selection alone
# ---------------------------------------------------------------------------
def _small_context(table, dt):
    """A context whose table or selection is what counts: any head will do."""
    d = table.shape[1]
    w = [torch.zeros((16, 3 * d), dtype=dt, device=DEV), torch.zeros((1, 16), dtype=dt, device=DEV)]
    return B.Context(dtype=B.AIF_F32 if dt == torch.float32 else B.AIF_BF16, table=table, d_user=d, d_attn=d, n_heads=1, max_seq_len=8,
                     layer_dims=[3 * d, 16, 1], weights=w, cross_mode=B.AIF_CROSS_NONE, max_candidates=256, max_users=64)


def _update_inputs(c, seed):
    g, dt = _gen(seed), _dt(c)
    return (_normal(g, (c["items"], c["d"]), dt), torch.randperm(c["items"], device=DEV, generator=g)[:c["rows"]].to(torch.int32),
            _normal(g, (c["rows"], c["d"]), dt))


def _prepare_update(c, seed):
    table, ids, rows = _update_inputs(c, seed)
    return dict(run=_run_update, ctx=_small_context(table, _dt(c)), table=table, ids=ids, rows=rows)


def _run_update(s):
    s["ctx"].aif_update_rows(s["ids"], s["rows"])
    return s["table"]


def _exact_update(c, seed):
    table, ids, rows = _update_inputs(c, seed)
    return table.index_copy_(0, ids.long(), rows)


def _topk_inputs(c, seed):
    return _normal(_gen(seed), (c["lists"], c["n"]), torch.float32, 0.3)


def _prepare_topk(c, seed):
    z = _topk_inputs(c, seed)
    return dict(run=_run_topk, ctx=_small_context(torch.zeros((64, 64), device=DEV), torch.float32), lists=list(z), k=c["k"],
                idx=torch.zeros((c["lists"], c["k"]), dtype=torch.int32, device=DEV), val=torch.zeros((c["lists"], c["k"]), device=DEV))


def _run_topk(s):
    s["ctx"].aif_topk(s["lists"], s["k"], s["idx"], s["val"])
    return {"best": s["val"], "positions": s["idx"]}


def _exact_topk(c, seed):
    v, at = torch.sort(_topk_inputs(c, seed), dim=1, descending=True, stable=True)
    more = max(0, c["k"] - c["n"])
    v, at = v[:, :c["k"]], at[:, :c["k"]].to(torch.int32)
    return {"best": torch.cat([v, v.new_full((c["lists"], more), -math.inf)], 1), "positions": torch.cat([at, at.new_full((c["lists"], more), -1)], 1)}


# ---------------------------------------------------------------------------
_PREPARE = dict(score=_prepare_score, user=_prepare_user, lsh=_prepare_lsh, update=_prepare_update, topk=_prepare_topk)
_EXACT = dict(score=_exact_score, user=_exact_user, lsh=_exact_lsh, update=_exact_update, topk=_exact_topk)


def prepare(case, seed):
    return _PREPARE[case["path"]](case, seed)


def run(state):
    return state["run"](state)


def exact(case, seed):
    return _EXACT[case["path"]](case, seed)


def work(case):
    if case["path"] == "score":
        return _work_score(case)
    if case["path"] == "user":
        return _work_user(case)
    if case["path"] == "lsh":
        return _work_lsh(case)
    if case["path"] == "update":
        return {"bytes": case["rows"] * (4 + 2 * case["d"] * (4 if case["dtype"] == "f32" else 2)), "flops": 0}
    return {"bytes": case["lists"] * (4 * case["n"] + 8 * case["k"]), "flops": 0}


def tolerance(case):
    """About four times what the path is off from 64 bits over the ranges above."""
    if case["path"] in ("update", "topk"):
        return "exact"                                  # rows are copied, logits only compared
    if case["path"] == "lsh":
        return {"rel": 1e-6, "max": 2e-5, "differ": 0.0}         # fp32 sums (seen: 4e-8); the counts are whole numbers
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4, "differ": 0.01}        # fp32 sums (seen: 7e-7); neighbours among the best may swap
    if case["path"] == "user":
        return {"rel": 8e-3, "max": 0.1}                # outputs stored in bf16 (seen: 1.8e-3)
    return {"rel": 1.5e-2, "max": 0.1}                  # bf16 weights, activations and attention (seen: 3.4e-3)
