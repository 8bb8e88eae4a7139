"""The work that is timed: retrieval calls as a user's program makes them, over
the sizes of this repository's configurations (20K x 128 up to 8.8M x 768) and
generic ones around them.

Kinds of work, one entry point of the framework each:

* ``dense``: open a query batch on an index, read its first ranks, close it
  (``pvs_open``, ``pvs_next``, ``pvs_close``).  ``pages`` > 1 reads on in pages
  that double, as a fusion or a client that pages through results does.
  ``deleted`` > 0 reads a snapshot taken after that share of rows was deleted.
* ``build``: quantise a segment of new rows that lie on the GPU and answer the
  first query batch on it (``pvs_build``, then as above, ``pvs_free``).
* ``sparse``: rank a batch of sparse queries with the posting work on the GPU
  (``pbm_gpu_open``, ``pbm_gpu_next``, ``pbm_gpu_close``).
* ``hybrid``: the ordered Top-20 of both channels (``eahr_topk``).

Rows are clustered unit vectors, documents draw half of their tokens from a
Zipf law and half from their cluster's topic terms, queries are drawn like rows
and take four of their cluster's topic terms: the recipe of the package's
``datagen``, drawn here with torch on the GPU so that inputs are quick to make.
"""
import math

import numpy as np
import torch

from paper_2608_07152_amd import eahr

DEV = "cuda"
STD = 0.5            # noise of a row around its centre
VOCAB, TOPIC, DOC_LEN, Q_TERMS, ZIPF = 30_000, 200, 60.0, 4, 1.1
K1, B_LEN = 0.9, 0.4
RANGE = 4096         # documents per block-max range
K = 20


def listed():
    return [
        # the smallest request: one query on a small collection, where launches, copies and waits are all there is
        {"name": "dense_20k_b1", "kind": "dense", "n": 20_000, "d": 128, "B": 1, "m": 20, "pages": 1, "deleted": 0.0},
        # a few queries on a collection of odd size and dimension, a tenth of its rows deleted
        {"name": "dense_300k_d100_b5_deleted", "kind": "dense", "n": 300_007, "d": 100, "B": 5, "m": 100, "pages": 1, "deleted": 0.1},
        # a small batch on the 1M x 384 collection
        {"name": "dense_1m_b16", "kind": "dense", "n": 1_000_000, "d": 384, "B": 16, "m": 100, "pages": 1, "deleted": 0.0},
        # a full batch on it, a re-ranker's thousand candidates each
        {"name": "dense_1m_b256_m1000", "kind": "dense", "n": 1_000_000, "d": 384, "B": 256, "m": 1000, "pages": 1, "deleted": 0.0},
        # one request on the 8.8M x 768 passage collection: the codes are streamed for one query
        {"name": "dense_passage_b1", "kind": "dense", "n": 8_800_000, "d": 768, "B": 1, "m": 1000, "pages": 1, "deleted": 0.0},
        # the headline batch on it
        {"name": "dense_passage_b256", "kind": "dense", "n": 8_800_000, "d": 768, "B": 256, "m": 100, "pages": 1, "deleted": 0.0},
        # a dimension that is neither 384 nor 768, a batch that fills no power of two
        {"name": "dense_2m_d1024_b100", "kind": "dense", "n": 2_000_000, "d": 1024, "B": 100, "m": 200, "pages": 1, "deleted": 0.0},
        # resumed reading on a snapshot with deletes: pages of 640, 1280, ... 40960 ranks
        {"name": "pages_4m_b64_deleted", "kind": "dense", "n": 4_000_000, "d": 768, "B": 64, "m": 640, "pages": 7, "deleted": 0.1},
        # a segment of new rows becomes searchable
        {"name": "build_200k_d768", "kind": "build", "n": 200_000, "d": 768, "B": 8, "m": 100},
        # the sparse channel of a batch on the GPU
        {"name": "sparse_1m_b256", "kind": "sparse", "n": 1_000_000, "B": 256, "m": 1000},
        # one hybrid request, and a batch of them
        {"name": "hybrid_1m_b1", "kind": "hybrid", "n": 1_000_000, "d": 384, "B": 1, "w_dense": 1, "sparse": "pbm"},
        {"name": "hybrid_2m_d768_b256", "kind": "hybrid", "n": 2_000_000, "d": 768, "B": 256, "w_dense": 1, "sparse": "pbm"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng):
    # the usual embedding sizes, and any other
    return rng.choice([128, 384, 768, 768, 1024]) if rng.random() < 0.6 else _log(rng, 64, 1100)


def draw(rng):
    """One more case of the ranges above, never dearer than the dearest listed one."""
    kind = rng.choice(["dense", "dense", "dense", "dense", "build", "sparse", "hybrid"])
    if kind == "dense":
        d = _dim(rng)
        n = min(_log(rng, 20_000, 8_800_000), 8_800_000 * 768 // max(d, 768))
        pages = rng.choice([1, 1, 1, rng.randint(2, 7)])
        B = _log(rng, 1, 256 if pages == 1 else 64)
        return {"kind": kind, "n": n, "d": d, "B": B, "m": min(_log(rng, 10, 1000), n // (2 << pages)), "pages": pages,
                "deleted": rng.choice([0.0, 0.0, 0.1])}
    if kind == "build":
        return {"kind": kind, "n": _log(rng, 20_000, 400_000), "d": _dim(rng), "B": _log(rng, 1, 64), "m": _log(rng, 10, 1000)}
    if kind == "sparse":
        return {"kind": kind, "n": _log(rng, 20_000, 1_000_000), "B": _log(rng, 1, 256), "m": _log(rng, 10, 1000)}
    return {"kind": kind, "n": _log(rng, 20_000, 2_000_000), "d": min(_dim(rng), 768), "B": _log(rng, 1, 256),
            "w_dense": rng.choice([1, 2]), "sparse": rng.choice(["pbm", "pbm", "pbm_gpu"])}


# ------------------------------------------------------------------ inputs
def _centers(case):
    return max(32, min(4096, case["n"] // 1000))


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 16 + stream) % (1 << 62))
    return g


def _rows(centers, labels, g):
    """normalize(centre + noise), drawn in chunks of rows."""
    n, d = labels.numel(), centers.shape[1]
    x = torch.empty(n, d, device=DEV)
    for r in range(0, n, 1 << 19):
        lab = labels[r:r + (1 << 19)]
        v = torch.randn(lab.numel(), d, device=DEV, generator=g).mul_(STD).add_(centers[lab])
        torch.div(v, v.norm(dim=1, keepdim=True), out=x[r:r + lab.numel()])
    return x


def _labels(case, seed):
    c = _centers(case)
    g = _gen(seed, 0)
    return (torch.randint(0, c, (case["n"],), device=DEV, generator=g),
            torch.randint(0, c, (case["B"],), device=DEV, generator=g))


def _dense_inputs(case, seed):
    """(rows, queries, ids deleted before the snapshot)."""
    lab, qlab = _labels(case, seed)
    centers = torch.randn(_centers(case), case["d"], device=DEV, generator=_gen(seed, 1))
    x = _rows(centers, lab, _gen(seed, 2))
    q = _rows(centers, qlab, _gen(seed, 3))
    gone = int(case.get("deleted", 0.0) * case["n"])
    ids = torch.randperm(case["n"], device=DEV, generator=_gen(seed, 4))[:gone]
    return x, q, ids


def _sparse_inputs(case, seed):
    """(term_ptr, docs, impacts) on the GPU and the queries' terms [B, 4]."""
    n, c = case["n"], _centers(case)
    lab, qlab = _labels(case, seed)
    g = _gen(seed, 5)
    topics = torch.rand(c, VOCAB, device=DEV, generator=g).topk(TOPIC, dim=1).indices
    perm = torch.randperm(VOCAB, device=DEV, generator=g)
    p = torch.arange(1, VOCAB + 1, device=DEV, dtype=torch.float64).pow(-ZIPF)
    cdf = (p.cumsum(0) / p.sum()).float()
    dl = torch.poisson(torch.full((n,), DOC_LEN, device=DEV), generator=g).clamp_(min=1).long()
    doc = torch.repeat_interleave(torch.arange(n, device=DEV), dl)
    t = doc.numel()
    zipf = perm[torch.searchsorted(cdf, torch.rand(t, device=DEV, generator=g)).clamp_(max=VOCAB - 1)]
    topic = topics[lab[doc], torch.randint(0, TOPIC, (t,), device=DEV, generator=g)]
    term = torch.where(torch.rand(t, device=DEV, generator=g) < 0.5, zipf, topic)
    key, tf = torch.unique(term * n + doc, return_counts=True)   # term-major, documents ascending
    term, doc = key // n, key % n
    df = torch.bincount(term, minlength=VOCAB)
    term_ptr = torch.zeros(VOCAB + 1, dtype=torch.int64, device=DEV)
    term_ptr[1:] = df.cumsum(0)
    idf = torch.log(1 + (n - df.double() + 0.5) / (df.double() + 0.5))
    norm = K1 * (1 - B_LEN + B_LEN * dl.double() / dl.double().mean())
    tf = tf.double()
    imp = (idf[term] * tf / (tf + norm[doc])).float()
    pick = torch.rand(case["B"], TOPIC, device=DEV, generator=g).topk(Q_TERMS, dim=1).indices
    return term_ptr, doc.int(), imp, topics[qlab[:, None], pick]


def _sparse_host(case, seed):
    """The sparse index and the queries, in host memory."""
    term_ptr, doc, imp, terms = _sparse_inputs(case, seed)
    index = eahr.pbm_build(term_ptr.cpu().numpy(), doc.cpu().numpy(), imp.cpu().numpy(), case["n"], RANGE)
    ones = np.ones(Q_TERMS, dtype=np.float32)
    return index, [(t, ones) for t in np.sort(terms.cpu().numpy(), axis=1).astype(np.int32)]


# ------------------------------------------------------------------- the work
def prepare(case, seed):
    """What the program holds before the call: the indexes, and the queries
    (the dense ones on the GPU, where an encoder leaves them)."""
    s = {"case": case}
    if case["kind"] in ("sparse", "hybrid"):
        s["pbm"], s["terms"] = _sparse_host(case, seed)
        if case["kind"] == "sparse" or case["sparse"] == "pbm_gpu":
            eahr.pbm_upload(s["pbm"])
    if case["kind"] == "build":
        s["x"], s["q"], _ = _dense_inputs(case, seed)
    elif case["kind"] != "sparse":
        x, s["q"], gone = _dense_inputs(case, seed)
        s["index"], s["epoch"] = eahr.pvs_build(x), 0
        if gone.numel():
            eahr.pvs_delete(s["index"], gone.cpu().numpy())
            s["epoch"] = eahr.pvs_snapshot(s["index"])
    return s


def _read(index, epoch, q, m, pages):
    st = eahr.pvs_open(index, q, epoch)
    ids, scores = [], []
    for p in range(pages):
        i, sc, _, _ = eahr.pvs_next(st, m << p)
        ids.append(i)
        scores.append(sc)
    eahr.pvs_close(st)
    return {"ids": ids, "scores": scores}


def run(state):
    case = state["case"]
    if case["kind"] == "dense":
        return _read(state["index"], state["epoch"], state["q"], case["m"], case["pages"])
    if case["kind"] == "build":
        index = eahr.pvs_build(state["x"])
        out = _read(index, 0, state["q"], case["m"], 1)
        eahr.pvs_free(index)
        return out
    if case["kind"] == "sparse":
        st = eahr.pbm_gpu_open(state["pbm"], state["terms"])
        got = eahr.pbm_gpu_next(st, case["m"])
        eahr.pbm_gpu_close(st)
        return {"ids": np.concatenate([g[0] for g in got]), "scores": np.concatenate([g[1] for g in got])}
    ids, count, _, stats = eahr.eahr_topk(state["index"], state["pbm"], state["q"], state["terms"], K=K,
                                          w_dense=case["w_dense"], sparse_generator=case["sparse"])
    return {"ids": ids, "count": count,
            "depths": np.array([[s["dense_depth"], s["sparse_depth"]] for s in stats], dtype=np.int64)}


def _postings(case):
    """About how many postings the batch's terms have."""
    in_cluster = case["n"] / _centers(case) * (1 - (1 - 0.5 / TOPIC) ** DOC_LEN)
    return case["B"] * Q_TERMS * (in_cluster + case["n"] * 0.5 * DOC_LEN / VOCAB)


def work(case):
    """The codes and their three floats once, the returned ranks' float32 rows
    once, the postings of the queries' terms once, the results."""
    n, d, B = case["n"], case.get("d", 0), case["B"]
    if case["kind"] == "sparse":
        return {"bytes": 8 * _postings(case) + 12 * B * case["m"], "flops": 2 * _postings(case)}
    ranks = B * (K if case["kind"] == "hybrid" else case["m"] * ((1 << case.get("pages", 1)) - 1))
    nbytes = n * (d + 12) + n / 8 + 4 * d * B + ranks * (4 * d + 12)
    if case["kind"] == "build":
        nbytes += 4 * n * d + 4 * n * d     # the rows read, and kept
    if case["kind"] == "hybrid":
        nbytes += 8 * _postings(case)
    return {"bytes": nbytes, "flops": 2 * n * d * B}


def tolerance(case):
    """Scores are float32 sums of up to 1100 products (measured against 64 bits:
    2-norm 8e-8, largest 1.2e-6), impacts float32 sums of four.  Another order
    of summation also swaps neighbours of a ranking: 0.05 % to 0.4 % of the ids
    of a first page differ from the 64-bit ranking, 2 % of 80,000 ranks."""
    return {"rel": 3e-7, "max": 5e-6, "differ": 0.01 if case["kind"] in ("dense", "build") else 0.002}


# --------------------------------------------------------------------- 64 bits
def _exact_dense(case, seed):
    """(ids, scores) of the first ranks of every query in float64."""
    x, q, gone = _dense_inputs(case, seed)
    total = case["m"] * ((1 << case.get("pages", 1)) - 1)
    alive = torch.ones(case["n"], dtype=torch.bool, device=DEV)
    alive[gone] = False
    q = q.double().T.contiguous()
    best_s = best_i = None
    for r in range(0, case["n"], 1 << 19):
        s = (x[r:r + (1 << 19)].double() @ q).T
        s = s.masked_fill(~alive[r:r + (1 << 19)], -math.inf)
        top = s.topk(min(total, s.shape[1]), dim=1)
        i = top.indices + r
        s = top.values
        if best_s is not None:
            s, i = torch.cat([best_s, s], 1), torch.cat([best_i, i], 1)
        top = s.topk(min(total, s.shape[1]), dim=1)
        best_s, best_i = top.values, i.gather(1, top.indices)
    return best_i, best_s


def _exact_sparse(case, seed):
    term_ptr, doc, imp, terms = _sparse_inputs(case, seed)
    ids, scores = [], []
    for t in terms.tolist():
        s = torch.zeros(case["n"], dtype=torch.float64, device=DEV)
        for k in t:
            a, b = int(term_ptr[k]), int(term_ptr[k + 1])
            s[doc[a:b].long()] += imp[a:b].double()
        top = s.topk(min(case["m"], int((s > 0).sum())))
        ids.append(top.indices)
        scores.append(top.values)
    return torch.cat(ids), torch.cat(scores)


def exact(case, seed):
    if case["kind"] == "hybrid":
        return None      # whole numbers only
    if case["kind"] == "sparse":
        return {"ids": None, "scores": _exact_sparse(case, seed)[1]}
    s = _exact_dense(case, seed)[1]
    cuts = [case["m"] << p for p in range(case.get("pages", 1))]
    return {"ids": None, "scores": [v.contiguous() for v in s.split(cuts, dim=1)]}
