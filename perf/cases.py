"""The workloads whose speed matters, as calls of the public entry points.

Every case scores words of a phoneme-encoded dictionary against each other (or
against query words).  The sizes and laws are those of the benchmark
configurations in ``synth`` and ``bench.py``; ``draw`` spreads further cases
over the same ranges.  A case is a dict of plain values:

kind      what the program asks for
          ``triangle``  scores of a range of pair indices, written to device memory
          ``topk``      every word's k best neighbours, with or without the histogram
          ``query``     the k best dictionary words of each query word
          ``edges``     the pairs of a weight slice, their graph, and an ego network
          ``batched``   the triangles of several dictionaries in one call
n         words of the dictionary (for ``batched`` the dictionary count is 8)
law       ``zipf``: 40 symbols, Zipf(1.1), lengths clip(Poisson(mean), 1, lmax),
          +1 / -1 / gap -1 (the paper's scoring);
          ``uniform``: 64 symbols, lengths 1..lmax, a symmetric 64 x 64
          similarity matrix in [-3, 3] with diagonal +3, gap -2
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2509_01654_amd as nw

_DTYPES = {"int8": torch.int8, "int16": torch.int16}
_BATCHED_SIZES = (1000, 3000, 10000, 20000, 40000, 60000, 80000, 100000)
_BATCHED_LMAX = tuple(int(round(8 + 40 * v / 7)) for v in range(8))
_ZIPF_ALPHABET, _UNIFORM_ALPHABET = 40, 64
_TILE = 1 << 28     # pairs of a chunk of a triangle that goes past device memory


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # a small dictionary, the whole triangle at once: latency and launches count
        _triangle("triangle_2k", 2000, "zipf", 7.0, 20, "int8"),
        # the ordinary full triangle that still fits in device memory
        _triangle("triangle_50k", 50000, "zipf", 7.0, 20, "int8"),
        # phonetic similarity matrix, wider scores, longer words
        _triangle("triangle_matrix_20k", 20000, "uniform", 0.0, 25, "int16"),
        # one restartable chunk from the middle of a triangle that does not fit
        _triangle("triangle_chunk_200k", 200000, "zipf", 8.0, 32, "int8", chunk=0.4),
        # words past the register-row limit (phrases, transcribed sentences)
        _triangle("triangle_long_6k", 6000, "uniform", 0.0, 255, "int16"),
        # the headline workload: the paper's 600,000 words
        _topk("topk_600k", 600000, "zipf", 8.0, 32, 32, True),
        # a small dictionary's neighbour lists alone
        _topk("topk_20k", 20000, "zipf", 7.0, 20, 16, False),
        # neighbour lists and histogram under a similarity matrix
        _topk("topk_matrix_30k", 30000, "uniform", 0.0, 31, 32, True),
        # one lookup in the full dictionary: what an interactive user waits for
        _query("query_1_of_600k", 600000, "zipf", 8.0, 32, 16, 1),
        # a batch of lookups, as the server gathers them under load
        _query("query_256_of_200k", 200000, "zipf", 8.0, 32, 16, 256),
        # graph export: a slice of normalised weights, its graph and an ego network
        _edges("edges_100k", 100001, "zipf", 8.0, 32, True, 60, 100),
        # several dictionaries with one similarity matrix, planned once and replayed
        dict(name="batched_8", kind="batched", scale=0.25, planned=True),
    ]


def draw(rng):
    kind = rng.choice(["triangle", "triangle", "topk", "query", "edges", "batched"])
    law = rng.choice(["zipf", "zipf", "uniform"])
    form = rng.choice(["whole", "whole", "chunk", "long"])
    if kind == "edges" or (kind == "triangle" and form == "chunk"):
        law = "zipf"
    mean = round(rng.uniform(6.0, 9.0), 2) if law == "zipf" else 0.0
    lmax = rng.randint(18, 36) if law == "zipf" else rng.randint(8, 48)
    if kind == "triangle":
        dtype = rng.choice(["int8", "int16"]) if law == "zipf" else "int16"
        if form == "long":
            return _triangle("", _odd(rng, 1000, 8000), "uniform", 0.0, rng.randint(49, 255), "int16")
        if form == "chunk":
            return _triangle("", _odd(rng, 40000, 300000), law, mean, lmax, dtype, chunk=round(rng.random() * 0.8, 4))
        return _triangle("", _odd(rng, 300, 60000 if law == "zipf" else 30000), law, mean, lmax, dtype)
    if kind == "topk":
        return _topk("", _odd(rng, 1000, 200000 if law == "zipf" else 40000), law, mean, lmax, rng.choice([8, 16, 32]),
                     rng.random() < 0.5)
    if kind == "query":
        return _query("", _odd(rng, 20000, 600000), law, mean, lmax, rng.choice([8, 16, 32]), _odd(rng, 1, 400))
    if kind == "edges":
        lo, hi = rng.choice([(60, 100), (70, 100), (80, 100)])
        return _edges("", _odd(rng, 2000, 200000), law, mean, lmax, True, lo, hi)
    return dict(kind="batched", scale=round(math.exp(rng.uniform(math.log(0.02), math.log(0.4))), 4),
                planned=rng.random() < 0.5)


def _odd(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _case(name, **kw):
    if name:
        kw["name"] = name
    return kw


def _triangle(name, n, law, mean, lmax, dtype, chunk=-1.0):
    # chunk < 0: the whole triangle; otherwise one chunk starting at that share of it
    return _case(name, kind="triangle", n=n, law=law, mean=mean, lmax=lmax, dtype=dtype, chunk=chunk)


def _topk(name, n, law, mean, lmax, k, hist):
    return _case(name, kind="topk", n=n, law=law, mean=mean, lmax=lmax, k=k, hist=hist)


def _query(name, n, law, mean, lmax, k, queries):
    return _case(name, kind="query", n=n, law=law, mean=mean, lmax=lmax, k=k, queries=queries)


def _edges(name, n, law, mean, lmax, normalised, lo, hi):
    return _case(name, kind="edges", n=n, law=law, mean=mean, lmax=lmax, normalised=normalised, lo=lo, hi=hi)


# --------------------------------------------------------------------------- inputs
def _lengths(rng, n, law, mean, lmax):
    if law == "zipf":
        return np.clip(rng.poisson(mean, size=n), 1, lmax).astype(np.int64)
    return rng.integers(1, lmax + 1, size=n).astype(np.int64)


def _words(seed, n, law, mean, lmax):
    """(symbols uint8, offsets uint64) of n words, drawn from the seed alone."""
    rng = np.random.default_rng(seed)
    lengths = _lengths(rng, n, law, mean, lmax)
    total = int(lengths.sum())
    if law == "zipf":
        p = np.arange(1, _ZIPF_ALPHABET + 1, dtype=np.float64) ** -1.1
        symbols = np.searchsorted(np.cumsum(p / p.sum())[:-1], rng.random(total), side="right")
    else:
        symbols = rng.integers(0, _UNIFORM_ALPHABET, size=total)
    offsets = np.zeros(n + 1, dtype=np.uint64)
    np.cumsum(lengths, out=offsets[1:])
    return symbols.astype(np.uint8), offsets


def _similarity(law):
    """(similarity matrix int64, gap): what the scoring of a law means."""
    if law == "zipf":
        return 2 * np.eye(_ZIPF_ALPHABET, dtype=np.int64) - 1, -1
    rng = np.random.default_rng(4)
    m = np.zeros((_UNIFORM_ALPHABET, _UNIFORM_ALPHABET), dtype=np.int64)
    iu = np.triu_indices(_UNIFORM_ALPHABET, k=1)
    m[iu] = rng.integers(-3, 4, size=iu[0].shape[0])
    m = m + m.T
    np.fill_diagonal(m, 3)
    return m, -2


def _scoring(law):
    if law == "zipf":
        return nw.Scoring(alphabet=_ZIPF_ALPHABET, match=1, mismatch=-1, gap=-1)
    m, gap = _similarity(law)
    return nw.Scoring(alphabet=_UNIFORM_ALPHABET, gap=gap, submat=m.astype(np.int8))


def _range(case):
    pairs = case["n"] * (case["n"] - 1) // 2
    if case["chunk"] < 0:
        return 0, pairs
    begin = int(pairs * case["chunk"])
    return begin, min(pairs, begin + _TILE)


def _bins(case):
    """(lowest score, number of scores) of words of lmax symbols."""
    sim, gap = _similarity(case["law"])
    lo, hi = case["lmax"] * min(int(sim.min()), gap, 0), case["lmax"] * max(int(sim.max()), 0)
    return lo, hi - lo + 1


def _edge_cap(case):
    # about 25 times the pairs the slices of these laws hold
    return max(4096, case["n"] * case["n"] // 4000)


def _batched_shapes(case):
    return [(max(2, int(round(n * case["scale"]))), lmax) for n, lmax in zip(_BATCHED_SIZES, _BATCHED_LMAX)]


# --------------------------------------------------------------------------- the calls
def prepare(case, seed):
    kind = case["kind"]
    if kind == "batched":
        vocabs = [nw.Vocab(*_words(seed * 16 + v, n, "uniform", 0.0, lmax), _scoring("uniform"))
                  for v, (n, lmax) in enumerate(_batched_shapes(case))]
        outs = [torch.empty(max(1, v.num_pairs), dtype=torch.int16, device="cuda") for v in vocabs]
        plan = nw.Batch(vocabs, dtype=torch.int16, class_width=0, use_graph=True, outs=outs) if case["planned"] else None
        return dict(case=case, vocabs=vocabs, outs=outs, plan=plan)
    vocab = nw.Vocab(*_words(seed, case["n"], case["law"], case["mean"], case["lmax"]), _scoring(case["law"]))
    st = dict(case=case, vocab=vocab)
    if kind == "triangle":
        begin, end = _range(case)
        st["out"] = torch.empty(end - begin, dtype=_DTYPES[case["dtype"]], device="cuda")
    elif kind == "topk":
        n, k = case["n"], case["k"]
        st["ws"] = torch.empty(vocab.topk_workspace_bytes(k), dtype=torch.uint8, device="cuda")
        st["out"] = (torch.empty((n, k), dtype=torch.int16, device="cuda"),
                     torch.empty((n, k), dtype=torch.int32, device="cuda"),
                     None)
        if case["hist"]:
            # bin 0 is the lowest score words of lmax symbols can reach; the
            # bounds of this dictionary's own longest word lie inside
            first, bins = _bins(case)
            st["hist"] = torch.zeros(bins, dtype=torch.int64, device="cuda")
            lo, hi = vocab.bounds
            st["out"] = (*st["out"][:2], st["hist"][lo - first:hi + 1 - first])
    elif kind == "query":
        nq, k = case["queries"], case["k"]
        st["queries"] = _words(seed + 1000003, nq, case["law"], case["mean"], case["lmax"])
        st["ws"] = torch.empty(vocab.query_workspace_bytes(nq, k), dtype=torch.uint8, device="cuda")
        st["out"] = (torch.empty((nq, k), dtype=torch.int16, device="cuda"),
                     torch.empty((nq, k), dtype=torch.int32, device="cuda"))
    else:
        cap = _edge_cap(case)
        st["out"] = (torch.empty(cap, dtype=torch.int32, device="cuda"),
                     torch.empty(cap, dtype=torch.int32, device="cuda"),
                     torch.empty(cap, dtype=torch.int16, device="cuda"))
        st["rows"] = tuple(torch.empty_like(t) for t in st["out"])
        st["count"] = torch.empty(1, dtype=torch.int64, device="cuda")
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batched":
        if state["plan"] is not None:
            return state["plan"].run()
        return nw.all_pairs_scores_batched(state["vocabs"], dtype=torch.int16, outs=state["outs"])
    vocab = state["vocab"]
    if kind == "triangle":
        begin, end = _range(case)
        return vocab.all_pairs_scores(begin, end, dtype=_DTYPES[case["dtype"]], out=state["out"])
    if kind == "topk":
        sc, ix, _ = vocab.all_pairs_topk(case["k"], hist=case["hist"], ws=state["ws"], out=state["out"])
        return (sc, ix, state["hist"]) if case["hist"] else (sc, ix)
    if kind == "query":
        return vocab.query(*state["queries"], k=case["k"], ws=state["ws"], out=state["out"])
    # the edges come in no particular order: a program that stores the graph
    # sorts them row-major into its table, as the paper's edge-weight file is
    # written; the table's unused rows hold -1
    n = case["n"]
    i, j, s, _ = vocab.all_pairs_edges(case["lo"], case["hi"], normalised=case["normalised"], out=state["out"],
                                       count=state["count"])
    order = torch.argsort(i.long() * n + j)
    for column, values in zip(state["rows"], (i, j, s)):
        column.fill_(-1)
        column[:order.numel()] = values[order]
    row_ptr, adj = nw.graph_csr(n, i, j)
    return *state["rows"], row_ptr, nw.ego_network(row_ptr, adj, [0, n // 2], 3)


# --------------------------------------------------------------------------- work
def work(case):
    """Bytes read and written once, and 5 operations per cell of a pair's score
    matrix (two adds, two maxima, one similarity)."""
    kind = case["kind"]
    if kind == "batched":
        shapes = [(n, "uniform", 0.0, lmax) for n, lmax in _batched_shapes(case)]
        nbytes = cells = 0
        for n, law, mean, lmax in shapes:
            m1, _ = _moments(law, mean, lmax)
            pairs = n * (n - 1) // 2
            nbytes += int(n * (m1 + 8)) + 2 * pairs
            cells += int(pairs * m1 * m1)
        return dict(bytes=nbytes, flops=5 * cells)
    n = case["n"]
    m1, _ = _moments(case["law"], case["mean"], case["lmax"])
    words = int(n * (m1 + 8))
    if kind == "triangle":
        begin, end = _range(case)
        es = 1 if case["dtype"] == "int8" else 2
        return dict(bytes=words + (end - begin) * es, flops=int(5 * (end - begin) * m1 * m1))
    pairs = n * (n - 1) // 2
    if kind == "topk":
        return dict(bytes=words + 6 * n * case["k"], flops=int(5 * pairs * m1 * m1))
    if kind == "query":
        nq = case["queries"]
        return dict(bytes=words + int(nq * (m1 + 8)) + 6 * nq * case["k"], flops=int(5 * n * nq * m1 * m1))
    return dict(bytes=words + 12 * n, flops=int(5 * pairs * m1 * m1))


def _moments(law, mean, lmax):
    l = _lengths(np.random.default_rng(0), 20000, law, mean, lmax).astype(np.float64)
    return float(l.mean()), float((l * l).mean())


# --------------------------------------------------------------------------- exact values
def exact(case, seed):
    """The same outputs from the definition (Algorithm 1) in 64-bit integers."""
    kind = case["kind"]
    if kind == "batched":
        shapes = _batched_shapes(case)
        if sum(n * (n - 1) // 2 * lmax * lmax for n, lmax in shapes) > _EXACT_CELLS:
            return None
        return [_triangle_exact(*_words(seed * 16 + v, n, "uniform", 0.0, lmax), "uniform", 0, n * (n - 1) // 2)
                for v, (n, lmax) in enumerate(shapes)]
    n, law, lmax = case["n"], case["law"], case["lmax"]
    if kind == "query":
        nq, k = case["queries"], case["k"]
        if n * nq * lmax * lmax > _EXACT_CELLS:
            return None
        D, Dl = _padded(*_words(seed, n, law, case["mean"], lmax))
        Q, Ql = _padded(*_words(seed + 1000003, nq, law, case["mean"], lmax))
        score = torch.empty((nq, k), dtype=torch.int64)
        index = torch.empty((nq, k), dtype=torch.int64)
        for q in range(nq):
            s = _pair_scores(Q[q:q + 1].expand(n, -1), Ql[q:q + 1].expand(n), D, Dl, law)
            score[q], index[q] = _best(s, torch.arange(n, device=s.device), k)
        return score, index
    begin, end = _range(case) if kind == "triangle" else (0, n * (n - 1) // 2)
    if (end - begin) * lmax * lmax > _EXACT_CELLS or n > 20000:
        return None
    symbols, offsets = _words(seed, n, law, case["mean"], lmax)
    tri = _triangle_exact(symbols, offsets, law, begin, end)
    if kind == "triangle":
        return tri
    iu = torch.from_numpy(np.stack(np.triu_indices(n, k=1)))
    if kind == "topk":
        full = torch.full((n, n), -(1 << 40), dtype=torch.int64)
        full[iu[0], iu[1]] = tri
        full[iu[1], iu[0]] = tri
        score = torch.empty((n, case["k"]), dtype=torch.int64)
        index = torch.empty((n, case["k"]), dtype=torch.int64)
        for u in range(n):
            j = torch.cat((torch.arange(u), torch.arange(u + 1, n)))
            score[u], index[u] = _best(full[u][j], j, case["k"])
        if not case["hist"]:
            return score, index
        first, bins = _bins(case)
        return score, index, torch.bincount(tri - first, minlength=bins)
    l = torch.from_numpy(np.diff(offsets.astype(np.int64)))
    m = torch.maximum(l[iu[0]], l[iu[1]]).clamp(min=1)
    keep = (100 * tri >= case["lo"] * m) & (100 * tri <= case["hi"] * m)
    i, j, s = iu[0][keep], iu[1][keep], tri[keep]
    rows = [torch.full((_edge_cap(case),), -1, dtype=torch.int64) for _ in range(3)]
    for column, values in zip(rows, (i, j, s)):
        column[:values.numel()] = values
    row_ptr = torch.zeros(n + 1, dtype=torch.int64)
    row_ptr[1:] = torch.cumsum(torch.bincount(torch.cat((i, j)), minlength=n), 0)
    dist = torch.full((n,), -1, dtype=torch.int64)
    dist[[0, n // 2]] = 0
    for hop in range(1, 4):
        front = dist == hop - 1
        reach = torch.zeros(n, dtype=torch.bool)
        reach[j[front[i]]] = True
        reach[i[front[j]]] = True
        dist[reach & (dist < 0)] = hop
    return *rows, row_ptr, dist


_EXACT_CELLS = 2_000_000_000


def _padded(symbols, offsets):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    l = np.diff(offsets.astype(np.int64))
    out = np.zeros((l.shape[0], max(1, int(l.max()))), dtype=np.int64)
    rows = np.repeat(np.arange(l.shape[0]), l)
    cols = np.arange(symbols.shape[0]) - np.repeat(offsets[:-1].astype(np.int64), l)
    out[rows, cols] = symbols
    return torch.from_numpy(out).to(dev), torch.from_numpy(l).to(dev)


def _pair_scores(A, la, B, lb, law):
    """Algorithm 1 of every pair (A[p], B[p]), a row of the score matrix at a time."""
    sim, gap = _similarity(law)
    sim = torch.from_numpy(sim).to(A.device)
    P, LA, LB = A.shape[0], int(la.max()), int(lb.max())
    row = [torch.full((P,), gap * j, dtype=torch.int64, device=A.device) for j in range(LB + 1)]
    out = torch.zeros(P, dtype=torch.int64, device=A.device)

    def read(i):
        done = la == i
        table = torch.stack([r[done] for r in row], 1)
        out[done] = table.gather(1, lb[done][:, None])[:, 0]

    read(0)
    for i in range(1, LA + 1):
        diag, row[0] = row[0], torch.full_like(row[0], gap * i)
        for j in range(1, LB + 1):
            up = row[j]
            row[j] = torch.maximum(diag + sim[A[:, i - 1], B[:, j - 1]], torch.maximum(up, row[j - 1]) + gap)
            diag = up
        read(i)
    return out


def _triangle_exact(symbols, offsets, law, begin, end):
    W, l = _padded(symbols, offsets)
    n = W.shape[0]
    iu = np.triu_indices(n, k=1)
    out = torch.empty(end - begin, dtype=torch.int64)
    step = 1 << 19
    for b in range(begin, end, step):
        e = min(end, b + step)
        i = torch.from_numpy(iu[0][b:e]).to(W.device)
        j = torch.from_numpy(iu[1][b:e]).to(W.device)
        out[b - begin:e - begin] = _pair_scores(W[i], l[i], W[j], l[j], law).cpu()
    return out


def _best(score, index, k):
    """The k best of (score descending, index ascending), padded with (-32768, -1)."""
    order = torch.argsort(-score * (1 << 32) + index)[:k]
    s = torch.full((k,), -32768, dtype=torch.int64)
    x = torch.full((k,), -1, dtype=torch.int64)
    s[:order.numel()] = score[order].cpu()
    x[:order.numel()] = index[order].cpu()
    return s, x
