"""Threshold edges by the plane kernels where their launches are cut: column steps
dealt to several workgroups (17,000 words), row groups dealt to several (words of
one length), ranges that cut blocks, dense slices that fill the queues, and
capacities below the count.  Against the oracle, as sets."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _matrix(A):
    return oracle.sim_matrix(A, submat=synth.random_submat(A, seed=4))


def _load(scheme, A, v):
    import paper_2509_01654_amd as nw
    if scheme == "plain":
        return nw.Vocab(v.symbols, v.offsets, nw.Scoring(A, 1, -1, -1)), oracle.sim_matrix(A, 1, -1), -1
    return nw.Vocab(v.symbols, v.offsets, nw.Scoring(A, submat=synth.random_submat(A, seed=4), gap=-2)), _matrix(A), -2


def _check(dv, v, sim, gap, lo, hi, i0, i1, caps=(None,)):
    ei, ej, es = oracle.edges(v.symbols, v.offsets, sim, gap, lo, hi, normalised=True, idx_begin=i0, idx_end=i1)[:3]
    want = np.stack([ei, ej, es]).astype(np.int64)
    want = want[:, np.lexsort((want[1], want[0]))]
    for cap in caps:
        c = None if cap is None else int(cap * want.shape[1])
        i, j, s, count = dv.all_pairs_edges(lo, hi, normalised=True, idx_begin=i0, idx_end=i1, cap=c)
        assert count == want.shape[1]
        got = np.stack([i.cpu().numpy(), j.cpu().numpy(), s.cpu().numpy()]).astype(np.int64)
        got = got[:, np.lexsort((got[1], got[0]))]
        if c is None or c >= count:
            np.testing.assert_array_equal(got, want)
        else:
            assert got.shape[1] == c and set(map(tuple, got.T.tolist())) <= set(map(tuple, want.T.tolist()))


@pytest.mark.parametrize("scheme,A", [("plain", 40), ("matrix", 64)])
@pytest.mark.parametrize("n,lmax", [(17000, 14), (33000, 9)])
def test_edges_of_large_blocks(scheme, A, n, lmax):
    """Blocks of 1,024 and 2,048 words: a few rows, cut inside rows, dense and sparse slices."""
    v = synth.uniform_vocab(n, seed=n, alphabet=A, min_len=0, max_len=lmax)
    dv, sim, gap = _load(scheme, A, v)
    start = lambda u: u * (2 * n - u - 1) // 2
    for a, b in ((start(0), start(1)), (start(1000) + 17, start(1050) + 999), (start(n - 900) + 3, start(n - 2)),
                 (start(n // 2) + 5, start(n // 2) + 6)):
        print(f"[gpu case] edges {scheme} {n} words, pairs {a}..{b}", flush=True)
        _check(dv, v, sim, gap, 40, 100, a, b, (None, 0.3))
        _check(dv, v, sim, gap, -1000, 1000, a, min(b, a + 40000))


@pytest.mark.parametrize("scheme,A", [("plain", 4), ("matrix", 64)])
@pytest.mark.parametrize("n,lo,hi", [(31, 6, 6), (300, 24, 24), (2300, 24, 24), (700, 48, 48), (1500, 44, 48)])
def test_edges_of_few_lengths(scheme, A, n, lo, hi):
    v = synth.uniform_vocab(n, seed=n + lo, alphabet=A, min_len=lo, max_len=hi)
    dv, sim, gap = _load(scheme, A, v)
    pairs = n * (n - 1) // 2
    print(f"[gpu case] edges {scheme} {n} words of {lo}..{hi}", flush=True)
    _check(dv, v, sim, gap, 20, 100, 0, pairs, (None, 0.5))
    _check(dv, v, sim, gap, -1000, 1000, pairs // 3 + 1, min(pairs, pairs // 3 + 150001))
