"""The work the search library is measured on, through its public entry points.

Every corpus and query set is synthetic and drawn on the GPU from the seed: Zipf(1.1) or
uniform term ids without repeats inside a row, lognormal(0, 0.8) or uniform weights, row
lengths around the mean of the setting.  The sizes are those of ``synth/workloads.py`` (the
SPLADE-FULL, AntSparse and RANDOM shapes, the exact and the differentiation settings) and of
the serving leg of ``bench.py``, with smaller and ragged ones beside them.

A case is a dict of plain values:

kind     search (Alg. 4), coarse (Alg. 2), serve (the request loop), score (pair scores with
         their gradient), build (index construction in device memory)
docs, vocab, doc_nnz, terms     the corpus: terms "zipf" (lognormal values) or "uniform"
alpha, vn, window, dtype        the index: mass-ratio pruning (vn 0) or vn entries a document
queries, query_nnz, spread      the queries: mean length, or lengths uniform over 5 to
                                2 query_nnz - 5 where spread is set
k, gamma, beta, host            the search: results, rerank pool, query pruning, queries
                                handed over in host memory
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2509_08395_amd as sindi

DEV = "cuda"
_ROWS = 250_000  # rows drawn at a time


def _case(kind, docs, queries, **kw):
    c = {"kind": kind, "docs": docs, "vocab": 30_522, "doc_nnz": 120, "terms": "zipf",
         "alpha": 0.5, "vn": 0, "window": 100_000, "dtype": "f16", "queries": queries,
         "query_nnz": 30, "spread": False, "k": 50, "gamma": 500, "beta": 1.0, "host": False}
    c.update(kw)
    return c


def listed():
    return [
        # One query against a small exact index (no pruning, one window): an embedded lookup
        # or a test fixture; nothing but latency.
        _case("search", 10_000, 1, name="one-10k", alpha=1.0, window=10_000, dtype="f32", k=10,
              gamma=10),
        # One query against the SPLADE-FULL-sized index, from host memory as it arrives: what
        # an interactive search waits for.
        _case("search", 8_800_000, 1, name="one-8.8m", doc_nnz=125, query_nnz=35, host=True),
        # A ragged handful of long and short queries with query pruning: a reranker's or a
        # multi-query retriever's call on a mid-sized collection.
        _case("search", 300_007, 37, name="few-300k", query_nnz=64, spread=True, beta=0.8, k=10,
              dtype="bf16", host=True),
        # The pruned FP32 setting: 1,000 queries evaluated over 1M documents.
        _case("search", 1_000_000, 1_000, name="eval-1m-f32", dtype="f32"),
        # The headline batch evaluation: 7,000 queries over 8.8M documents, FP16 postings.
        _case("search", 8_800_000, 7_000, name="bulk-8.8m", doc_nnz=125, query_nnz=35),
        # The fastest setting at full recall: strong document and query pruning, small pool.
        _case("search", 8_800_000, 7_000, name="bulk-8.8m-fast", doc_nnz=125, query_nnz=35,
              alpha=0.2, gamma=200, beta=0.8),
        # Short queries over a large vocabulary (AntSparse shape): most lists hold few postings.
        _case("search", 1_000_000, 1_000, name="short-1m", vocab=250_000, doc_nnz=40, query_nnz=6,
              alpha=0.85, window=50_000),
        # Uniformly random terms and values (RANDOM shape), BF16 postings: no heavy terms.
        _case("search", 1_000_000, 1_000, name="random-1m-bf16", vocab=30_000, terms="uniform",
              query_nnz=50, dtype="bf16"),
        # Exact top-100 without pruning or rerank: the candidates of a training step.
        _case("coarse", 1_000_000, 256, name="exact-1m", vocab=250_002, doc_nnz=180, query_nnz=40,
              alpha=1.0, dtype="f32", k=100, gamma=100),
        # The training step on those candidates: scores and the gradients of query and document
        # values through autograd.
        _case("score", 1_000_000, 256, name="train-1m", vocab=250_002, doc_nnz=180, query_nnz=40,
              alpha=1.0, dtype="f32", k=100, gamma=100),
        # A burst of requests of 5 to 200 terms and mixed k at the server: peak load.
        _case("serve", 2_200_000, 1_500, name="serve-2.2m", doc_nnz=125, query_nnz=102,
              spread=True, k=100, beta=0.8),
        # Index construction from a corpus in device memory, then the first queries on it: a
        # collection that is rebuilt as its encoder changes.
        _case("build", 1_000_000, 16, name="build-1m", doc_nnz=125, query_nnz=35),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "coarse", "serve", "score", "build"])
    shape = rng.choice([("zipf", 30_522, rng.uniform(90, 140), rng.uniform(4, 70)),
                        ("zipf", 30_522, rng.uniform(90, 140), rng.uniform(20, 45)),
                        ("zipf", 250_000, rng.uniform(30, 60), rng.uniform(4, 9)),
                        ("uniform", rng.choice([10_000, 30_000, 100_000]), rng.uniform(90, 130),
                         rng.uniform(30, 60))])
    terms, vocab, doc_nnz, query_nnz = shape
    docs = _spread(rng, 10_000, 2_000_000) if kind == "search" else _spread(rng, 100_000, 1_200_000)
    queries = _spread(rng, 1, 7_000)
    if kind in ("serve", "coarse", "score"):
        queries = _spread(rng, 64, 1_500 if kind == "serve" else 600)
    c = _case(kind, docs, queries, vocab=vocab, doc_nnz=int(doc_nnz), terms=terms,
              query_nnz=max(4, int(query_nnz)), spread=query_nnz > 12 and rng.random() < 0.4,
              alpha=rng.choice([0.2, 0.3, 0.4, 0.5, 0.5, 0.7, 0.85]),
              window=rng.choice([20_000, 50_000, 100_000, 250_000]),
              dtype=rng.choice(["f16", "f16", "bf16", "f32"]), k=rng.choice([1, 10, 50, 77, 100]),
              gamma=rng.choice([100, 200, 333, 500, 1_000]), beta=rng.choice([1.0, 1.0, 0.8, 0.7]),
              host=kind == "search" and rng.random() < 0.3)
    if kind in ("search", "build") and rng.random() < 0.2:
        c["vn"] = rng.randint(8, 45)
    if kind in ("coarse", "score"):
        c.update(alpha=1.0, dtype="f32", beta=1.0, spread=c["spread"] and kind == "coarse")
    if kind == "coarse":
        c["gamma"] = c["k"]
    if kind == "build":
        c["queries"] = rng.randint(1, 64)
    return c


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=64)
def _terms(terms, vocab, mean):
    """Term probabilities (float64 [vocab]) and the draws a row needs so that its distinct
    terms are `mean` on average."""
    p = np.full(vocab, 1.0 / vocab) if terms == "uniform" else np.arange(1, vocab + 1) ** -1.1
    p /= p.sum()
    lo, hi = float(mean), 64.0 * mean
    for _ in range(50):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if -np.expm1(-mid * p).sum() < mean else (lo, mid)
    return p, lo


@functools.lru_cache(maxsize=64)
def _cdf(terms, vocab, mean):
    return torch.from_numpy(np.cumsum(_terms(terms, vocab, mean)[0])).float().to(DEV)


def _rows(gen, n, case, mean, spread):
    """Rows as (lengths int64 [n], term ids int32, values float32): the points of a Poisson
    process, already ascending, mapped through the inverse distribution of the terms, repeats
    dropped."""
    p, draws = _terms(case["terms"], case["vocab"], mean)
    cdf = _cdf(case["terms"], case["vocab"], mean)
    rate = torch.full((n, 1), draws, device=DEV)
    if spread:  # lengths from 5 to 2 mean - 5
        rate = (torch.rand((n, 1), device=DEV, generator=gen) * (2 * mean - 10) + 5) * (draws / mean)
    top = float(draws * (2 if spread else 1))
    width = int(top + 6 * math.sqrt(top) + 8)
    u = torch.empty((n, width), device=DEV).exponential_(generator=gen).cumsum_(1)
    ok = u < rate
    t = torch.searchsorted(cdf, u.div_(rate), out_int32=True).clamp_(max=case["vocab"] - 1)
    ok[:, 1:] &= t[:, 1:] != t[:, :-1]
    ids = t[ok]
    if case["terms"] == "uniform":
        val = torch.rand(ids.shape, device=DEV, generator=gen).clamp_(min=1e-3)
    else:
        val = torch.randn(ids.shape, device=DEV, generator=gen).mul_(0.8).exp_()
    return ok.sum(1), ids, val


def _corpus_chunks(case, seed):
    gen = torch.Generator(DEV).manual_seed(2 * seed + 1)
    for r in range(0, case["docs"], _ROWS):
        yield _rows(gen, min(_ROWS, case["docs"] - r), case, case["doc_nnz"], False)


def _csr(parts, case, mean):
    lens, ids, val = (torch.cat(x) for x in zip(*parts))
    if case["kind"] == "score":  # gradients of one size for every seed: the surplus, spread
        nnz, total = ids.shape[0], lens.shape[0] * mean  # over the rows, is left out
        drop = nnz - int(0.99 * total - 5 * math.sqrt(total))
        at = torch.arange(drop, device=DEV) * nnz // drop
        keep = torch.ones(nnz, dtype=torch.bool, device=DEV)
        keep[at] = False
        row = torch.searchsorted(torch.cumsum(lens, 0), at, right=True)
        lens, ids, val = lens.index_add(0, row, -torch.ones_like(row)), ids[keep], val[keep]
    indptr = torch.zeros(lens.shape[0] + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=indptr[1:])
    return sindi.DeviceCsr(indptr, ids, val, case["vocab"])


def _queries(case, seed):
    gen = torch.Generator(DEV).manual_seed(2 * seed)
    return _csr([_rows(gen, case["queries"], case, case["query_nnz"], case["spread"])], case,
                case["query_nnz"])


def _candidates(case, seed):
    """Candidate ids of a training step and the gradient of its loss by their scores: hard
    negatives shared by several queries, as searches return them, then some of any document."""
    gen = torch.Generator(DEV).manual_seed(7919 * seed + 5)
    pool = torch.randint(0, case["docs"], (4 * case["k"],), device=DEV, generator=gen)
    shape = (case["queries"], case["k"])
    pick = pool[torch.randint(0, pool.shape[0], shape, device=DEV, generator=gen)]
    far = torch.randint(0, case["docs"], shape, device=DEV, generator=gen)
    cand = torch.where(torch.rand(shape, device=DEV, generator=gen) < 0.3, pick, far)
    return cand, torch.randn(shape, device=DEV, generator=gen) / case["k"]


def _request_ks(case, seed):
    gen = np.random.default_rng(seed)
    return gen.choice(sorted({max(1, case["k"] // 10), max(1, case["k"] // 2), case["k"]}),
                      case["queries"]).astype(np.int32)


class _Host:
    """A CSR in host memory."""

    def __init__(self, q):
        self.indptr, self.indices, self.values = (t.cpu().numpy() for t in (q.indptr, q.indices, q.values))
        self.n_cols = q.n_cols


def _index(case, corpus):
    prune = dict(prune="vnp", vn=case["vn"]) if case["vn"] else dict(alpha=case["alpha"])
    return sindi.Index(corpus, window=case["window"], value_dtype=case["dtype"], gpu_build=True, **prune)


def prepare(case, seed):
    q = _queries(case, seed)
    corpus = _csr(list(_corpus_chunks(case, seed)), case, case["doc_nnz"])
    st = {"case": case, "queries": _Host(q) if case["host"] or case["kind"] == "serve" else q}
    if case["kind"] == "build":
        st["corpus"] = corpus
        return st
    st["index"] = _index(case, corpus)
    if case["kind"] == "serve":
        st["server"] = sindi.Server(st["index"], k_max=case["k"], gamma=max(case["gamma"], case["k"]),
                                    beta=case["beta"])
        st["ks"] = _request_ks(case, seed)
        st["arrival"] = np.zeros(case["queries"])
    if case["kind"] == "score":
        st["cand"], st["grad"] = _candidates(case, seed)
        st["query_values"] = q.values.requires_grad_(True)
        st["doc_values"] = corpus.values.requires_grad_(True)
    return st


def run(st):
    case, q = st["case"], st["queries"]
    gamma = max(case["gamma"], case["k"])
    if case["kind"] == "search":
        return st["index"].search(q, case["k"], gamma=gamma, beta=case["beta"])
    if case["kind"] == "coarse":
        return st["index"].search_coarse(q, case["k"], beta=case["beta"])
    if case["kind"] == "serve":
        ids, scores, _ = st["server"].replay(q, st["ks"], st["arrival"])
        return ids, scores
    if case["kind"] == "score":
        s = sindi.SindiScore.apply(st["query_values"], st["doc_values"], st["index"], q.indptr,
                                   q.indices, st["cand"])
        gq, gx = torch.autograd.grad(s, (st["query_values"], st["doc_values"]), st["grad"])
        return s.detach(), gq, gx
    st["index"] = index = _index(case, st["corpus"])
    info = index.info()
    ids, scores = index.search(q, case["k"], gamma=gamma, beta=case["beta"])
    return ids, scores, info["n_postings"], info["n_tiles"]


# ------------------------------------------------------------------ floors
def work(case):
    """Expected bytes and operations of one pass: every posting list that a query names read
    once, every pooled document's row once, queries and results once; one multiply-add per
    posting of a query's term and per common term of a scored pair."""
    nd, nq, k = case["docs"], case["queries"], case["k"]
    pd, dd = _terms(case["terms"], case["vocab"], case["doc_nnz"])
    _, dq = _terms(case["terms"], case["vocab"], case["query_nnz"])
    in_doc, in_query = -np.expm1(-dd * pd), -np.expm1(-dq * pd)
    if case["vn"]:
        kept = min(1.0, case["vn"] / case["doc_nnz"])
    elif case["alpha"] >= 1.0:
        kept = 1.0
    elif case["terms"] == "uniform":  # the top share s of uniform values holds s (2 - s) of the mass
        kept = 1.0 - math.sqrt(1.0 - case["alpha"])
    else:  # lognormal: Phi(Phi^-1(alpha) - sigma)
        lo, hi = -9.0, 9.0
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if 0.5 * math.erfc(-mid / math.sqrt(2)) < case["alpha"] else (lo, mid)
        kept = 0.5 * math.erfc(-(lo - 0.8) / math.sqrt(2))
    vb = 4 if case["dtype"] == "f32" else 2
    corpus = nd * case["doc_nnz"] * 8 + nd * 8
    lists = nd * kept * (2 + vb)
    query = nq * (case["query_nnz"] * 8 + 8)
    if case["kind"] == "score":
        rows = nd * -math.expm1(-nq * k * 0.7 / nd) + min(nd, 4 * k)
        pairs = nq * k * float((in_doc * in_query).sum())
        return {"bytes": 2 * rows * case["doc_nnz"] * 8 + 4 * nd * case["doc_nnz"] + 2 * query + 12 * nq * k,
                "flops": 6 * pairs}
    touched = float((in_doc * -np.expm1(nq * np.log1p(-in_query * (1 - 1e-12)))).sum())
    postings = nd * kept * float((in_doc * in_query).sum())
    pool = 0 if case["kind"] == "coarse" else max(case["gamma"], k)
    rows = nd * -math.expm1(-nq * pool / nd)
    b = lists * touched + rows * case["doc_nnz"] * 8 + query + nq * k * 12
    f = 2 * nq * (postings + pool * float((in_doc * in_query).sum()))
    if case["kind"] == "build":  # the corpus is copied, its lists are written
        b += 2 * corpus + lists * case["doc_nnz"]
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ 64 bits
def _order_by_size(lens, val):
    """Entries row by row, largest |value| first (ties by term id), and every entry's row."""
    row = torch.repeat_interleave(torch.arange(lens.shape[0], device=DEV), lens)
    o = torch.sort(val.abs(), descending=True, stable=True).indices
    return o[torch.sort(row[o], stable=True).indices], row


def _keep(lens, val, alpha, vn):
    """The entries that pruning keeps: the shortest prefix by size that reaches alpha of the
    row's mass, or vn entries."""
    if alpha >= 1.0 and not vn:
        return torch.ones_like(val, dtype=torch.bool)
    o, row = _order_by_size(lens, val)
    first = torch.cumsum(lens, 0) - lens
    if vn:
        rank = torch.arange(val.shape[0], device=DEV) - first[row[o]]
        good = rank < vn
    else:
        before = torch.cumsum(val[o].double().abs(), 0) - val[o].double().abs()
        base = before[first.clamp(max=val.shape[0] - 1)]
        mass = torch.zeros(lens.shape[0], dtype=torch.float64, device=DEV).index_add_(0, row, val.double().abs())
        good = before - base[row[o]] < alpha * mass[row[o]]
    keep = torch.zeros_like(val, dtype=torch.bool)
    keep[o] = good
    return keep


def _dense(q, rows, vocab, keep=None):
    """Queries `rows` as a float64 [vocab, n] matrix."""
    a, b = int(q.indptr[rows[0]]), int(q.indptr[rows[-1] + 1])
    n = len(rows)
    lens = q.indptr[rows[0] + 1:rows[-1] + 2] - q.indptr[rows[0]:rows[-1] + 1]
    col = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    v = q.values[a:b].detach().double()
    if keep is not None:
        v = v * keep[a:b]
    d = torch.zeros((vocab, n), dtype=torch.float64, device=DEV)
    d[q.indices[a:b].long(), col] = v
    return d


def _products(lens, ids, val, dense):
    """float64 [rows, n] = the sparse rows times the dense matrix, 16,384 rows at a time."""
    out = torch.empty((lens.shape[0], dense.shape[1]), dtype=torch.float64, device=DEV)
    ends = [0] + torch.cumsum(lens, 0).tolist()
    step = 16_384
    for r in range(0, lens.shape[0], step):
        a, b = ends[r], ends[min(r + step, lens.shape[0])]
        part = lens[r:r + step]
        prod = val[a:b].double()[:, None] * dense[ids[a:b].long()]
        row = torch.repeat_interleave(torch.arange(part.shape[0], device=DEV), part)
        out[r:r + step] = torch.zeros((part.shape[0], dense.shape[1]), dtype=torch.float64,
                                      device=DEV).index_add_(0, row, prod)
    return out


_STORED = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _exact_search(case, seed):
    """Scores of Alg. 4 (or Alg. 2) in 64 bits: [queries, k], -inf past the corpus."""
    q, nq, k = _queries(case, seed), case["queries"], case["k"]
    coarse = case["kind"] == "coarse"
    qlens = q.indptr[1:] - q.indptr[:-1]
    qkeep = _keep(qlens, q.values, case["beta"], 0) if case["beta"] < 1.0 else None
    need = min(case["docs"], k if coarse else max(case["gamma"], k))
    blocks = [range(i, min(i + 64, nq)) for i in range(0, nq, 64)]
    best = [None] * len(blocks)
    for lens, ids, val in _corpus_chunks(case, seed):
        keep = _keep(lens, val, case["alpha"], case["vn"])
        row = torch.repeat_interleave(torch.arange(lens.shape[0], device=DEV), lens)
        klens = torch.zeros_like(lens).index_add_(0, row, keep.long())
        kids, kval = ids[keep], val[keep].to(_STORED[case["dtype"]])
        first = torch.cumsum(lens, 0) - lens
        for i, rows in enumerate(blocks):
            c = _products(klens, kids, kval, _dense(q, rows, case["vocab"], qkeep)).T.contiguous()
            c, d = torch.topk(c, min(need, c.shape[1]), dim=1)
            if coarse:
                s = c
            else:  # the pooled documents' full rows with the full queries
                full = _dense(q, rows, case["vocab"])
                n = lens[d.reshape(-1)]
                col = torch.repeat_interleave(torch.arange(n.shape[0], device=DEV), n)
                at = torch.arange(col.shape[0], device=DEV) - (torch.cumsum(n, 0) - n)[col] + first[d.reshape(-1)][col]
                p = val[at].double() * full[ids[at].long(), col // d.shape[1]]
                s = torch.zeros(n.shape[0], dtype=torch.float64, device=DEV).index_add_(0, col, p).reshape(d.shape)
            if best[i] is not None:
                c, s = torch.cat([best[i][0], c], 1), torch.cat([best[i][1], s], 1)
            c, at = torch.topk(c, min(need, c.shape[1]), dim=1)
            best[i] = (c, s.gather(1, at))
    out = torch.full((nq, k), -math.inf, dtype=torch.float64, device=DEV)
    for rows, (_, s) in zip(blocks, best):
        n = min(k, s.shape[1])
        out[rows[0]:rows[-1] + 1, :n] = torch.topk(s, n, dim=1).values
    return out


def _exact_score(case, seed):
    """Pair scores and their gradients in 64 bits."""
    q = _queries(case, seed)
    corpus = _csr(list(_corpus_chunks(case, seed)), case, case["doc_nnz"])
    cand, grad = _candidates(case, seed)
    x = corpus.values.double()
    s = torch.zeros(cand.shape, dtype=torch.float64, device=DEV)
    gq = torch.zeros(q.nnz, dtype=torch.float64, device=DEV)
    gx = torch.zeros_like(x)
    ptr, qptr = corpus.indptr, q.indptr.tolist()
    for b in range(case["queries"]):
        d = cand[b]
        n = ptr[d + 1] - ptr[d]
        col = torch.repeat_interleave(torch.arange(d.shape[0], device=DEV), n)
        at = torch.arange(col.shape[0], device=DEV) - (torch.cumsum(n, 0) - n)[col] + ptr[d][col]
        e = slice(qptr[b], qptr[b + 1])
        place = torch.full((case["vocab"],), -1, dtype=torch.int64, device=DEV)
        place[q.indices[e].long()] = torch.arange(qptr[b], qptr[b + 1], device=DEV)
        to = place[corpus.indices[at].long()]
        hit = to >= 0
        to, at, col = to[hit], at[hit], col[hit]
        g, qv = grad[b].double()[col], q.values.detach().double()[to]
        s[b].index_add_(0, col, qv * x[at])
        gq.index_add_(0, to, g * x[at])
        gx.index_add_(0, at, g * qv)
    return s, gq, gx


def exact(case, seed):
    if case["kind"] == "score":
        return _exact_score(case, seed)
    # about 20 seconds of products and selections
    if case["docs"] * case["queries"] * case["doc_nnz"] * (1.0 if case["alpha"] >= 1.0 else 0.3) > 3e11:
        return None
    s = _exact_search(case, seed)
    if case["kind"] == "serve":
        ks = torch.from_numpy(_request_ks(case, seed)).to(DEV)
        s = torch.where(torch.arange(case["k"], device=DEV) < ks[:, None], s, -math.inf)
    return (None, s, None, None) if case["kind"] == "build" else (None, s)
