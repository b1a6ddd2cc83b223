"""Kernels of dictionaries above 16,384 words, whose blocks hold 1,024 words and more,
in the forms that no other test reaches at that size: three planes, the packed
kernels (a weight above 7), and launches cut for few row lengths.  Also query batches
whose image is copied instead of carried as kernel arguments.  Against the oracle,
bit-exact."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PACKED = (4, -1, -2)   # a match weighs 8


def _report(name):
    print(f"[gpu case] {name}", flush=True)


def _load(kind, v):
    """(dictionary, similarity, gap) under three planes or packed."""
    import paper_2509_01654_amd as nw
    A = v.alphabet
    if kind == "matrix":
        S = synth.random_submat(A, seed=4)
        return nw.Vocab(v.symbols, v.offsets, nw.Scoring(A, submat=S, gap=-2)), oracle.sim_matrix(A, submat=S), -2
    match, mismatch, gap = PACKED if kind == "packed" else (1, -1, -1)
    return (nw.Vocab(v.symbols, v.offsets, nw.Scoring(A, match, mismatch, gap)), oracle.sim_matrix(A, match, mismatch), gap)


def _start(n, u):
    return u * (2 * n - u - 1) // 2


def _check_ranges(dv, v, sim, gap, ranges, dtype=torch.int16):
    """Every range into a buffer 1 .. 3 bytes past an aligned address, nothing written beside it."""
    import paper_2509_01654_amd as nw
    es = 2 if dtype == torch.int16 else 1
    for q, (a, b) in enumerate(ranges):
        shift = q % 4
        buf = torch.full(((b - a) * es + 16,), 0x55, dtype=torch.uint8, device="cuda")
        rc = nw._lib.nw_all_pairs_scores(dv._h, a, b, es, ctypes.c_void_p(buf.data_ptr() + shift),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == nw.NW_OK
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        got = host[shift:shift + (b - a) * es].copy().view(np.int16 if es == 2 else np.int8)
        np.testing.assert_array_equal(got.astype(np.int32), oracle.triangle(v.symbols, v.offsets, sim, gap, a, b),
                                      err_msg=f"pairs {a}..{b}")
        assert (host[:shift] == 0x55).all() and (host[shift + (b - a) * es:] == 0x55).all(), (a, b)


def _cuts(n):
    s = lambda u: _start(n, u)
    return [(s(0), s(1)), (s(1023) + 7, s(1025) + 3), (s(2047), s(2049)), (s(n // 3) + 100, s(n // 3 + 40) + 9),
            (s(n // 2) + 5, s(n // 2) + 6), (s(n - 1100) + 1, s(n - 1000)), (s(n - 60), s(n - 1))]


@pytest.mark.parametrize("kind", ["matrix", "packed"])
@pytest.mark.parametrize("n,lmax", [(17000, 25), (17000, 48), (33000, 14), (33000, 36)])
def test_triangle(kind, n, lmax):
    """Blocks of 1,024 and 2,048 words; matrix scores of up to 48 symbols need 16-bit
    staging, packed ones of 25 and 48 lie in and past the score-code window's pairs."""
    _report(f"triangle {kind} {n} words to {lmax}")
    v = synth.uniform_vocab(n, seed=n + lmax, alphabet=64 if kind == "matrix" else 40, min_len=0, max_len=lmax)
    dv, sim, gap = _load(kind, v)
    _check_ranges(dv, v, sim, gap, _cuts(n))
    out = dv.all_pairs_scores(dtype=torch.int16)
    torch.cuda.synchronize()
    for u in (0, 1023, 1024, 2048, n // 2, n - 1025, n - 2):
        a, b = _start(n, u), _start(n, u + 1)
        np.testing.assert_array_equal(out[a:b].cpu().numpy().astype(np.int32),
                                      oracle.triangle(v.symbols, v.offsets, sim, gap, a, b), err_msg=f"row {u}")
    rng = np.random.default_rng(n)
    i = rng.integers(0, n - 1, 200_000)
    j = i + 1 + (rng.random(i.size) * (n - 1 - i)).astype(np.int64)
    idx = i * (2 * n - i - 1) // 2 + (j - i - 1)
    np.testing.assert_array_equal(out[torch.from_numpy(idx).cuda()].cpu().numpy().astype(np.int32),
                                  oracle.pairs(v.symbols, v.offsets, sim, gap, i, j))


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_packed_triangle_any_alignment(shift):
    """The score-code triangle with a launch per row length: int8 at every byte."""
    _report(f"packed triangle shifted by {shift}")
    import paper_2509_01654_amd as nw
    v = synth.zipf_vocab(16500, seed=77, mean_len=7.0, max_len=20)
    dv, sim, gap = _load("packed", v)
    want = oracle.triangle(v.symbols, v.offsets, sim, gap, 0, _start(v.n, 2100))
    base = torch.full((dv.num_pairs + 8,), 99, dtype=torch.int8, device="cuda")
    dv.all_pairs_scores(dtype=torch.int8, out=base[shift:shift + dv.num_pairs])
    torch.cuda.synchronize()
    got = base[:want.size + shift].cpu().numpy().astype(np.int32)
    np.testing.assert_array_equal(got[shift:], want)
    assert (got[:shift] == 99).all() and (base[shift + dv.num_pairs:].cpu().numpy() == 99).all()
    _check_ranges(dv, v, sim, gap, [(12345, 3_000_001), (dv.num_pairs - 500_003, dv.num_pairs), (7, 8)], torch.int8)


@pytest.mark.parametrize("n,lmax,k", [(17000, 20, 16), (33000, 12, 32)])
def test_packed_topk(n, lmax, k):
    _report(f"packed top-{k} of {n} words")
    v = synth.zipf_vocab(n, seed=n, mean_len=7.0, min_len=0, max_len=lmax)
    dv, sim, gap = _load("packed", v)
    s, i, h = dv.all_pairs_topk(k)
    torch.cuda.synchronize()
    assert int(h.sum()) == n * (n - 1) // 2
    s, i = s.cpu().numpy().astype(np.int32), i.cpu().numpy()
    for r0 in (0, 1023, 2040, n // 2, n - 24):
        ws, wi, _ = oracle.topk_rows(v.symbols, v.offsets, sim, gap, k, r0=r0, r1=r0 + 24)
        np.testing.assert_array_equal(i[r0:r0 + 24], wi)
        np.testing.assert_array_equal(s[r0:r0 + 24], ws)


def test_packed_edges():
    n = 17000
    _report(f"packed edges of {n} words")
    v = synth.zipf_vocab(n, seed=5, mean_len=7.0, min_len=0, max_len=20)
    dv, sim, gap = _load("packed", v)
    for a, b in ((_start(n, 0), _start(n, 1)), (_start(n, 1000) + 9, _start(n, 1100) + 5), (_start(n, n - 500), _start(n, n - 1))):
        ei, ej, es = oracle.edges(v.symbols, v.offsets, sim, gap, 100, 400, normalised=True, idx_begin=a, idx_end=b)[:3]
        i, j, s, count = dv.all_pairs_edges(100, 400, normalised=True, idx_begin=a, idx_end=b)
        assert count == len(ei)
        assert sorted(zip(i.tolist(), j.tolist(), s.tolist())) == sorted(zip(map(int, ei), map(int, ej), map(int, es)))


@pytest.mark.parametrize("kind,n,lo,hi", [("plain", 2300, 24, 24), ("plain", 300, 30, 48), ("matrix", 4000, 24, 24),
                                          ("matrix", 9000, 1, 20), ("matrix", 3100, 12, 12), ("plain", 5000, 48, 48)])
def test_triangle_of_few_lengths_and_small_blocks(kind, n, lo, hi):
    """Launches cut down to one row group a workgroup, whole rows and rows listed inside blocks of 256 words."""
    _report(f"triangle {kind} {n} words of {lo}..{hi}")
    v = synth.uniform_vocab(n, seed=n, alphabet=64 if kind == "matrix" else 40, min_len=lo, max_len=hi)
    dv, sim, gap = _load(kind, v)
    pairs = n * (n - 1) // 2
    big = min(pairs, 6_500_000)   # (three planes take ranges of some millions of pairs)
    _check_ranges(dv, v, sim, gap, [(0, big), (pairs // 3 + 1, min(pairs, pairs // 3 + 1 + big)), (pairs - big + 3, pairs),
                                    (_start(n, n // 2) + 1, _start(n, n // 2 + 3) + 2)])


def test_batch_of_large_blocks_tiled():
    """The eight dictionaries of the batched workload at a quarter of their sizes, their
    own launches replayed as a graph and issued by one call."""
    import paper_2509_01654_amd as nw
    _report("batched, tiled form, up to 25,000 words")
    vocabs, S = synth.batched_configs(scale=0.25)
    sim = oracle.sim_matrix(64, submat=S)
    dvs = [nw.Vocab(v.symbols, v.offsets, nw.Scoring(64, submat=S, gap=-2)) for v in vocabs]
    b = nw.Batch(dvs, torch.int16, class_width=0, use_graph=True)
    for rep in range(2):
        for o in b.outs:
            o.fill_(-12345)
        torch.cuda.synchronize()
        outs = b.run()
        torch.cuda.synchronize()
    once = nw.all_pairs_scores_batched(dvs, dtype=torch.int16)
    torch.cuda.synchronize()
    rng = np.random.default_rng(3)
    for v, o, c in zip(vocabs, outs, once):
        n = v.n
        assert torch.equal(o[:n * (n - 1) // 2], c[:n * (n - 1) // 2])
        i = rng.integers(0, n - 1, 60_000)
        j = i + 1 + (rng.random(i.size) * (n - 1 - i)).astype(np.int64)
        idx = i * (2 * n - i - 1) // 2 + (j - i - 1)
        np.testing.assert_array_equal(o[torch.from_numpy(idx).cuda()].cpu().numpy().astype(np.int32),
                                      oracle.pairs(v.symbols, v.offsets, sim, -2, i, j))
    b.close()


@pytest.mark.parametrize("nq", [360, 420, 1500])
def test_query_batches_on_both_sides_of_the_copy(nq):
    """About 370 queries make an image of 24 KiB: below it goes up as kernel
    arguments, above by a copy.  Two calls in a row on one workspace."""
    import paper_2509_01654_amd as nw
    _report(f"{nq} queries")
    v = synth.zipf_vocab(3000, seed=50, mean_len=8.0, max_len=32)
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(v.alphabet, 1, -1, -1))
    sim = oracle.sim_matrix(v.alphabet, 1, -1)
    ws = torch.empty(dv.query_workspace_bytes(nq, 16), dtype=torch.uint8, device="cuda")
    batches = [synth.uniform_vocab(nq, seed=s, alphabet=40, min_len=0, max_len=48) for s in (1, 2)]
    got = [dv.query(q.symbols, q.offsets, 16, ws=ws) for q in batches]
    torch.cuda.synchronize()
    for q, (s, i) in zip(batches, got):
        ws_, wi = oracle.query(v.symbols, v.offsets, sim, -1, q.symbols, q.offsets, 16)
        np.testing.assert_array_equal(i.cpu().numpy(), wi)
        np.testing.assert_array_equal(s.cpu().numpy().astype(np.int32), ws_)
