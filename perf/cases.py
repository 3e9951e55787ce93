"""The work whose speed this repository tracks, one case per use of the library.

A user of this library holds a datastore of unit-norm token embeddings on the
GPU and asks, at every decode step, for the k best keys of B query embeddings
and their continuations.  The cases cover that use from the smallest datastore
to the largest that one index holds here, for the three key types, for one
query and for batches, exact, next-token-filtered, grouped by first token and
partitioned; the query-side transform and the draft packing that stand around
the search; and the two jobs that come before it, training the partitions and
building an index.

listed() are the cases themselves, draw() makes more of the same ranges.
prepare() makes what a program holds before the call, run() is one call,
exact() the same result in 64 bits from plain torch.
"""
import math

import torch

import paper_2502_15572_amd as dresd

DEV = "cuda:0"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
L = 10               # tokens a value holds
VOCAB = 32000
TOKEN_ZIPF = 1.1     # law of the tokens
HIDDEN = 4096        # width of the hidden states that the transform takes
CHUNK = 1 << 20


def listed():
    return [
        # A small session datastore, fp32 keys straight from the model: a call is all latency.
        {"name": "search_small_f32", "kind": "search", "dtype": "f32", "N": 16384, "d": 256,
         "B": 8, "k": 10, "filtered": False},
        # Keys at the hidden width of a 7B model, one sequence being decoded.
        {"name": "search_wide_bf16_b1", "kind": "search", "dtype": "bf16", "N": 1 << 20, "d": 4096,
         "B": 1, "k": 10, "filtered": False},
        # The same datastore under batched serving.
        {"name": "search_wide_bf16_b64", "kind": "search", "dtype": "bf16", "N": 1 << 20,
         "d": 4096, "B": 64, "k": 10, "filtered": False},
        # 256 principal components, a large serving batch.
        {"name": "search_10m_f16_b256", "kind": "search", "dtype": "f16", "N": 10_000_000,
         "d": 256, "B": 256, "k": 32, "filtered": False},
        # The largest datastore: 128 components, many drafts per query.
        {"name": "search_33m_f16_b128", "kind": "search", "dtype": "f16", "N": 1 << 25, "d": 128,
         "B": 128, "k": 100, "filtered": False},
        # Drafts must start with the model's next token; row count, width and batch all ragged.
        {"name": "filtered_ragged_f16_b13", "kind": "search", "dtype": "f16", "N": 2_999_999,
         "d": 100, "B": 13, "k": 30, "filtered": True},
        # One whole decode step of one sequence: hidden state -> query -> drafts, on the largest
        # datastore grouped by first token.
        {"name": "decode_step_33m_b1", "kind": "step", "dtype": "f16", "N": 1 << 25, "d": 128,
         "B": 1, "k": 100, "r": 10},
        # Approximate search of one query, the paper's own setting.
        {"name": "partitioned_33m_b1", "kind": "partitioned", "dtype": "f16", "N": 1 << 25,
         "d": 128, "B": 1, "k": 100, "P": 8192, "nprobe": 64},
        # Approximate search of a serving batch.
        {"name": "partitioned_33m_b128", "kind": "partitioned", "dtype": "f16", "N": 1 << 25,
         "d": 128, "B": 128, "k": 100, "P": 8192, "nprobe": 16},
        # Hidden states of a corpus to keys, one chunk of an index build.
        {"name": "transform_bulk", "kind": "transform", "M": 65536, "D": HIDDEN, "l": 128},
        # One k-means step over a training sample: new centroids from the last assignment, and
        # every row's nearest centroid among them.
        {"name": "train_partitions", "kind": "train", "dtype": "f16", "N": 524288, "d": 128,
         "P": 8192},
        # A datastore grouped by first token, from keys on the GPU to its first answer.
        {"name": "build_by_token_4m", "kind": "build", "dtype": "f16", "N": 1 << 22, "d": 128,
         "B": 4, "k": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "step", "partitioned",
                       "partitioned", "transform", "train", "build"])
    if kind == "transform":
        M, l = _log(rng, 1, 65536), _log(rng, 32, 1024)
        return {"kind": kind, "M": min(M, max(1, 65536 * 128 // l)), "D": rng.choice(
            [HIDDEN, _log(rng, 768, 4096)]), "l": l}
    dtype = rng.choice(["f16", "f16", "f16", "bf16", "bf16", "f32"])
    d = rng.choice([32, 64, 128, 256, 512, 1024, 2048, 4096, _log(rng, 32, 4096)])
    k = rng.choice([10, 16, 32, 100, _log(rng, 1, 100)])
    B = rng.choice([1, 1, 4, 8, _log(rng, 1, 256)])
    room = (1 << 33) // (d * SIZE[dtype])
    if kind == "search":
        if dtype == "f32" or d > 1024:   # the batches these keys are searched with
            B = min(B, 64)
        N = _log(rng, 16384, min(1 << 25, room))
        return {"kind": kind, "dtype": dtype, "N": N, "d": d, "B": B, "k": min(k, N),
                "filtered": rng.random() < 0.25}
    d = min(d, 512)
    if kind == "train":
        d = min(d, 256)
        N = _log(rng, 20000, 524288)
        return {"kind": kind, "dtype": dtype, "N": N, "d": d,
                "P": min(max(8, N // 64), 8192 * 128 // max(d, 128))}
    if kind == "build":
        return {"kind": kind, "dtype": dtype, "N": _log(rng, 65536, (1 << 22) * 128 // max(
            d, 128)), "d": d, "B": min(B, 8), "k": k}
    N = _log(rng, 200000, min(1 << 25, (1 << 33) // (d * SIZE[dtype])))
    if kind == "step":
        return {"kind": kind, "dtype": dtype, "N": N, "d": d, "B": min(B, 4), "k": k,
                "r": rng.choice([3, 10, 20])}
    P = min(8192, max(64, N // 4096))
    return {"kind": kind, "dtype": dtype, "N": N, "d": d, "B": min(B, 128), "k": k, "P": P,
            "nprobe": min(P, _log(rng, 4, 64))}


# ---- inputs ---------------------------------------------------------------------------------


def _gen(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + part)
    return g


def _unit(x):
    return x / x.norm(dim=1, keepdim=True)


def _clusters(case):
    return case.get("P") or max(16, min(8192, case["N"] // 256))


def _keys(case, seed):
    """Unit rows around cluster centres with per-cluster, per-dimension scales in [0.1, 1]."""
    N, d, C = case["N"], case["d"], _clusters(case)
    g = _gen(seed, 0)
    centres = torch.randn(C, d, device=DEV, generator=g)
    scales = torch.pow(10.0, -torch.rand(C, d, device=DEV, generator=g))
    owner = torch.randint(0, C, (N,), device=DEV, generator=g)
    keys = torch.empty(N, d, dtype=DT[case["dtype"]], device=DEV)
    step = max(1, (CHUNK * 256) // d)
    for a in range(0, N, step):
        o = owner[a:a + step]
        x = torch.randn(o.numel(), d, device=DEV, generator=g).mul_(scales[o]).add_(centres[o])
        keys[a:a + step] = _unit(x).to(keys.dtype)
    return keys, centres, owner


def _token_law():
    w = torch.arange(1, VOCAB + 1, dtype=torch.float64).pow(-TOKEN_ZIPF)
    return w / w.sum()


def _values(N, seed):
    g = _gen(seed, 1)
    cdf = torch.cumsum(_token_law(), 0).to(torch.float32).to(DEV)
    cont = torch.empty(N, L, dtype=torch.int32, device=DEV)
    for a in range(0, N, 4 * CHUNK):
        n = min(4 * CHUNK, N - a)
        u = torch.rand(n * L, device=DEV, generator=g)
        cont[a:a + n] = torch.searchsorted(cdf, u, out_int32=True).clamp_(
            max=VOCAB - 1).view(n, L)
    return cont


def _queries(keys, B, seed):
    """Stored rows seen again with noise, and the rows they come from."""
    g = _gen(seed, 2)
    src = torch.randint(0, keys.shape[0], (B,), device=DEV, generator=g)
    q = keys[src].to(torch.float32)
    return _unit(q + 0.1 * torch.randn(q.shape, device=DEV, generator=g)).contiguous(), src


def _affine(D, l, seed):
    """Datastore statistics and an orthonormal basis, as fitted offline."""
    g = _gen(seed, 3)
    mean = 0.5 * torch.randn(D, device=DEV, generator=g)
    var = torch.rand(D, device=DEV, generator=g) * 2.0 + 0.05
    W = torch.linalg.qr(torch.randn(D, max(l, 1), device=DEV, generator=g))[0].contiguous()
    return mean, var, W


def _inputs(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "transform":
        mean, var, W = _affine(case["D"], case["l"], seed)
        z = torch.randn(case["M"], case["D"], device=DEV, generator=_gen(seed, 4))
        s.update(mean=mean, var=var, W=W, x=z.mul_(var.sqrt()).add_(mean))
        return s
    s["keys"], s["centres"], s["owner"] = _keys(case, seed)
    if kind == "train":
        s.update(assign=s["owner"].to(torch.int32), centroids=_unit(s["centres"]).contiguous())
        return s
    s["cont"] = _values(case["N"], seed)
    s["q"], src = _queries(s["keys"], case["B"], seed)
    s["nt"] = s["cont"][src, 0].contiguous()
    if kind == "step":
        # hidden states whose projection is the query, with noise outside the basis
        mean, var, W = _affine(HIDDEN, case["d"], seed)
        z = s["q"] @ W.t().contiguous() + 0.01 * torch.randn(
            case["B"], HIDDEN, device=DEV, generator=_gen(seed, 4))
        s.update(mean=mean, var=var, W=W, x=(z * var.sqrt() + mean).contiguous())
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "search":
        s["index"] = dresd.Index(s["keys"], s["cont"])
    elif kind == "step":
        s["index"] = dresd.PartitionedIndex.by_first_token(s["keys"], s["cont"])
    elif kind == "partitioned":
        s["index"] = dresd.PartitionedIndex(s["keys"], s["cont"], _unit(s["centres"]).contiguous(),
                                            s["owner"].to(torch.int32))
    if "index" in s:     # an index holds its own copy; a program lets go of the tensors
        for name in ("keys", "cont", "centres", "owner"):
            del s[name]
    return s


# ---- the call -------------------------------------------------------------------------------


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "search":
        return s["index"].search(s["q"], case["k"],
                                 next_tok=s["nt"] if case["filtered"] else None)
    if kind == "partitioned":
        return s["index"].search(s["q"], case["k"], case["nprobe"])
    if kind == "step":
        y = dresd.transform(s["x"], s["mean"], s["var"], s["W"])
        idx, score, tok = s["index"].search_next_token(y, s["nt"], case["k"])
        drafts, count = dresd.pack_drafts(tok, case["r"], L)
        return y, idx, score, tok, drafts, count
    if kind == "transform":
        return dresd.transform(s["x"], s["mean"], s["var"], s["W"])
    if kind == "train":
        c = s["centroids"].clone()     # the update is in place
        counts = dresd.kmeans_update(s["keys"], s["assign"], c)
        assign, score = dresd.kmeans_assign(s["keys"], c, with_score=True)
        return c, counts, assign, score
    ix = dresd.PartitionedIndex.by_first_token(s["keys"], s["cont"])
    out = ix.search_next_token(s["q"], s["nt"], case["k"])
    ix.close()
    return out


# ---- what a pass cannot do without ----------------------------------------------------------


def work(case):
    kind = case["kind"]
    if kind == "transform":
        M, D, l = case["M"], case["D"], case["l"]
        return {"bytes": 4 * (M * D + 2 * D + D * l + M * l), "flops": 2 * M * D * l}
    N, d, es = case["N"], case["d"], SIZE[case["dtype"]]
    if kind == "train":
        P = case["P"]
        # the rows once for the sums and once against every new centroid
        return {"bytes": 2 * N * d * es + 4 * (2 * P * d + 3 * N + P), "flops": 2 * N * d * P}
    B, k = case["B"], case["k"]
    small = 4 * B * d + B * k * (12 + 8 * L)
    same = float(_token_law().pow(2).sum())   # share of the rows a query's next token keeps
    if kind == "search":
        if case["filtered"]:
            return {"bytes": N * d * es + 4 * N + 4 * B + small, "flops": 2 * N * d * B}
        return {"bytes": N * d * es + small, "flops": 2 * N * d * B}
    if kind == "partitioned":
        n = N * case["nprobe"] / case["P"]
        reach = N * (1.0 - (1.0 - case["nprobe"] / case["P"]) ** B)
        return {"bytes": int(reach * d * es + 4 * case["P"] * d + small),
                "flops": int(2 * d * B * (n + case["P"]))}
    if kind == "step":
        reach = min(N * same * B, N)
        return {"bytes": int(reach * d * es + 4 * (B * HIDDEN + 2 * HIDDEN + HIDDEN * d) + small
                             + 4 * B * case["r"] * L),
                "flops": int(2 * d * B * (N * same + HIDDEN))}
    # build: the keys and values read once and written once
    return {"bytes": int(2 * N * (d * es + 4 * L) + min(N * same * B, N) * d * es + small),
            "flops": int(2 * d * B * N * same)}


def tolerance(case):
    # Scores: 16-bit keys are searched with f16- or bf16-rounded query parts in larger batches.
    # Rows and tokens: neighbours in rank whose scores agree to rounding may trade places.
    kind = case["kind"]
    if kind == "transform":
        return {"rel": 4e-6}
    if kind == "train":
        # a row whose two best centroids score alike may go to the other one
        return {"rel": 2e-6, "differ": 1e-3}
    if kind == "search" and case["dtype"] == "f16" and case["B"] > 4:
        return {"rel": 4e-4, "differ": 0.01}
    return {"rel": 2e-6, "differ": 0.01}


# ---- 64 bits --------------------------------------------------------------------------------


def _top(keys, cont, q, k, rows=None, mask=None):
    """Top-k of every query over ``rows`` (all of them if None) that ``mask(rows)`` ([n, B], if
    given) keeps; (idx, score, tokens), padded with (-1, -inf, 0)."""
    B, n = q.shape[0], keys.shape[0] if rows is None else rows.numel()
    q = q.to(torch.float64).t().contiguous()
    best = torch.full((B, k), -math.inf, dtype=torch.float64, device=DEV)
    who = torch.full((B, k), -1, dtype=torch.int64, device=DEV)
    step = max(1, min((CHUNK * 128) // keys.shape[1], (CHUNK * 256) // B))
    for a in range(0, n, step):
        r = torch.arange(a, min(n, a + step), device=DEV) if rows is None else rows[a:a + step]
        x = (keys[a:a + step] if rows is None else keys[r]).to(torch.float64)
        sc = (x @ q).t()
        if mask is not None:
            sc = sc.masked_fill(~mask(r), -math.inf)
        v, j = torch.topk(sc, min(k, sc.shape[1]), dim=1)
        v, o = torch.topk(torch.cat([best, v], 1), k, dim=1)
        who = torch.cat([who, r[j]], 1).gather(1, o)
        best = v
    who = torch.where(best > -math.inf, who, torch.full_like(who, -1))
    tok = torch.where((who >= 0)[:, :, None], cont[who.clamp(min=0)],
                      torch.zeros((), dtype=cont.dtype, device=DEV))
    return who, best, tok


def _project(s):
    z = (s["x"].to(torch.float64) - s["mean"].to(torch.float64)) / torch.sqrt(
        s["var"].to(torch.float64) + 1e-5)
    y = z @ s["W"].to(torch.float64)
    return y / y.norm(dim=1, keepdim=True).clamp(min=1e-12)


def _nearest(x, c):
    c = c.to(torch.float64).t().contiguous()
    step = max(1, (CHUNK * 256) // c.shape[1])
    best = [(x[a:a + step].to(torch.float64) @ c).max(1) for a in range(0, x.shape[0], step)]
    return (torch.cat([b.indices for b in best]).to(torch.int32),
            torch.cat([b.values for b in best]))


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "transform":
        return _project(s)
    keys = s["keys"]
    if kind == "train":
        total = torch.zeros(s["centroids"].shape, dtype=torch.float64, device=DEV)
        total.index_add_(0, s["owner"], keys.to(torch.float64))
        norm = total.norm(dim=1, keepdim=True)
        c = torch.where(norm > 0, total / norm.clamp(min=1e-300),
                        s["centroids"].to(torch.float64))
        counts = torch.bincount(s["owner"], minlength=case["P"]).to(torch.int32)
        return (c, counts) + _nearest(keys, c)
    cont, q, nt, k = s["cont"], s["q"], s["nt"], case["k"]
    if kind == "search" and not case["filtered"]:
        return _top(keys, cont, q, k)
    first = cont[:, 0].contiguous()
    if kind == "partitioned":
        cent = _unit(s["centres"]).to(torch.float64)
        probe = torch.topk(q.to(torch.float64) @ cent.t().contiguous(), case["nprobe"], dim=1)[1]
        hit = torch.zeros(case["B"], case["P"], dtype=torch.bool, device=DEV)
        hit.scatter_(1, probe, True)
        parts = [_top(keys, cont, q[b:b + 1], k, rows=torch.nonzero(hit[b][s["owner"]]).view(-1))
                 for b in range(case["B"])]
        return tuple(torch.cat(p) for p in zip(*parts))
    y = None
    if kind == "step":
        y = _project(s)
        q = y
    parts = [_top(keys, cont, q[b:b + 1], k, rows=torch.nonzero(first == nt[b]).view(-1))
             for b in range(case["B"])]
    out = tuple(torch.cat(p) for p in zip(*parts))
    return (y,) + out + (None, None) if kind == "step" else out
