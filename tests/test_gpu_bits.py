"""GPU parity of the bit-plane kernels against the oracle (bit-exact).

The sizes are the edges of their layout: words of every length up to the
register-row limit of 48 (each length has its own code, most groups of 32 row
words mix lengths), empty words, dictionaries that leave padding slots and
half-filled groups, alphabets on both sides of a 32-symbol mask, and scorings on
both sides of every rule that picks 2 planes, 3 planes or the packed kernels.
Scores are integers: no tolerance.
"""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from synth import uniform_vocab, vocab_from_words, zipf_vocab

pytestmark = pytest.mark.gpu


def _nw():
    import torch
    import paper_2509_01654_amd as nw
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return nw, torch


def _matrix(alphabet, lo, hi, diag, seed=9):
    rng = np.random.default_rng(seed)
    m = np.triu(rng.integers(lo, hi + 1, size=(alphabet, alphabet)), 1)
    m = m + m.T
    np.fill_diagonal(m, diag)
    return m


# name: (alphabet, similarity matrix as scored by the oracle, gap, Scoring keywords)
def _scorings():
    out = {}
    for name, A, match, mismatch, gap in [
        ("plain", 40, 1, -1, -1),             # 2 planes
        ("plain_gap2", 33, -1, -3, -2),       # 2 planes, other bounds
        ("plain_gap0", 6, 3, 1, 0),           # 2 planes, no fill of short rows
        ("levenshtein", 32, 0, -1, -1),       # 3 planes, weights 2 and 1
        ("lcs", 3, 1, 0, 0),                  # 3 planes, weights 1 and 0, heavy ties
        ("negative_weights", 20, 2, -9, -2),  # 3 planes, mismatches weigh -5
        ("weight_8", 20, 4, -1, -2),          # packed kernels
    ]:
        out[name] = (A, oracle.sim_matrix(A, match, mismatch), gap, dict(match=match, mismatch=mismatch))
    for name, A, lo, hi, diag, gap in [("matrix_64", 64, -3, 3, 3, -2), ("matrix_65", 65, -2, 1, 3, -2),
                                       ("matrix_200", 200, -1, 0, 1, -1)]:
        m = _matrix(A, lo, hi, diag)
        out[name] = (A, m, gap, dict(submat=m))
    m = oracle.sim_matrix(40, 1, -1)
    out["plain_as_matrix"] = (40, m, -1, dict(submat=m))
    return out


SCORINGS = _scorings()


def _words(n, alphabet, lmax, seed=5):
    """n words of lengths 0 .. lmax, every length present, some words repeated."""
    rng = np.random.default_rng(seed)
    lengths = rng.integers(0, lmax + 1, size=n)
    lengths[: min(n, lmax + 1)] = np.arange(lmax + 1)[: min(n, lmax + 1)]
    words = [rng.integers(0, alphabet, size=l) for l in rng.permutation(lengths)]
    for i in range(0, n - 7, 50):
        words[i + 6] = words[i]
    return vocab_from_words(words, alphabet)


def _load(name, v):
    nw, torch = _nw()
    A, sim, gap, kw = SCORINGS[name]
    return nw.Vocab(v.symbols, v.offsets, nw.Scoring(alphabet=A, gap=gap, **kw), device="cuda:0"), sim, gap


@pytest.mark.parametrize("hist", [True, False])
@pytest.mark.parametrize("name", list(SCORINGS))
@pytest.mark.parametrize("n,lmax", [(333, 48), (257, 11)])
def test_topk_bits(name, n, lmax, hist):
    _, torch = _nw()
    v = _words(n, SCORINGS[name][0], lmax)
    dv, sim, gap = _load(name, v)
    k = 9
    sc, ix, h = dv.all_pairs_topk(k, hist=hist)
    torch.cuda.synchronize()
    ws, wi, wh = oracle.topk_rows(v.symbols, v.offsets, sim, gap, k, hist_range=dv.bounds)
    assert np.array_equal(sc.cpu().numpy().astype(np.int32), ws)
    assert np.array_equal(ix.cpu().numpy(), wi)
    if hist:
        assert np.array_equal(h.cpu().numpy().astype(np.uint64), wh)


@pytest.mark.parametrize("n", [2, 31, 33, 64, 65, 256, 17000])
def test_topk_bits_group_edges(n):
    """Groups and steps that end inside a block, and past the small-block rule."""
    _, torch = _nw()
    v = zipf_vocab(n, seed=n, mean_len=6.0, min_len=0, max_len=14)
    dv, sim, gap = _load("plain", v)
    sc, ix, h = dv.all_pairs_topk(5)
    torch.cuda.synchronize()
    for r0 in {0, max(0, n - 60), (n // 2) & ~31}:
        r1 = min(n, r0 + 60)
        ws, wi, _ = oracle.topk_rows(v.symbols, v.offsets, sim, gap, 5, r0=r0, r1=r1)
        assert np.array_equal(sc.cpu().numpy()[r0:r1].astype(np.int32), ws)
        assert np.array_equal(ix.cpu().numpy()[r0:r1], wi)
    assert int(h.sum()) == n * (n - 1) // 2


def _ranges(n, pairs, rng):
    """Whole triangle, single pairs, parts of one row, row ends, ranges over a few rows and over many."""
    start = lambda u: u * (2 * n - u - 1) // 2
    out = [(0, pairs), (0, 1), (pairs - 1, pairs), (start(3) + 2, start(3) + 9), (start(5), start(6)),
           (start(n // 2) + 1, start(n // 2 + 40) + 3)]
    for _ in range(4):
        a, b = sorted(rng.integers(0, pairs + 1, size=2).tolist())
        out.append((a, b))
    return out


@pytest.mark.parametrize("dtype", ["int8", "int16"])
@pytest.mark.parametrize("name", list(SCORINGS))
@pytest.mark.parametrize("n,lmax", [(333, 48), (530, 11), (140, 36)])
def test_triangle_bits(name, n, lmax, dtype):
    """Every range and output alignment (bytes before the first element) against the oracle."""
    nw, torch = _nw()
    v = _words(n, SCORINGS[name][0], lmax, seed=6)
    dv, sim, gap = _load(name, v)
    dt, es = (torch.int8, 1) if dtype == "int8" else (torch.int16, 2)
    if dtype == "int8" and not (dv.bounds[0] >= -128 and dv.bounds[1] <= 127):
        with pytest.raises(nw.NwError):
            dv.all_pairs_scores(dtype=dt)
        return
    want = oracle.triangle(v.symbols, v.offsets, sim, gap)
    pairs = want.size
    for q, (a, b) in enumerate(_ranges(n, pairs, np.random.default_rng(n))):
        shift = q % 4
        buf = torch.full(((b - a) * es + 16,), 0x55, dtype=torch.uint8, device="cuda:0")
        rc = nw._lib.nw_all_pairs_scores(dv._h, a, b, es, ctypes.c_void_p(buf.data_ptr() + shift),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == nw.NW_OK
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        got = host[shift:shift + (b - a) * es].copy().view(np.int8 if es == 1 else np.int16)
        assert np.array_equal(got.astype(np.int64), want[a:b]), (a, b, shift)
        assert (host[:shift] == 0x55).all() and (host[shift + (b - a) * es:] == 0x55).all(), (a, b, shift)


@pytest.mark.parametrize("n,lmax", [(17000, 14), (40000, 20), (33000, 30)])
def test_triangle_bits_windows(n, lmax):
    """Blocks of 1024, 2048 words and windows of 1024: a few rows, whole and cut, against the oracle."""
    _, torch = _nw()
    v = zipf_vocab(n, seed=n, mean_len=7.0, min_len=0, max_len=lmax)
    dv, sim, gap = _load("plain", v)
    start = lambda u: u * (2 * n - u - 1) // 2
    out = dv.all_pairs_scores(dtype=torch.int8)
    torch.cuda.synchronize()
    for u in (0, 1023, 1024, 2047, 2048, n // 2, n - 1025, n - 2):
        want = oracle.triangle(v.symbols, v.offsets, sim, gap, start(u), start(u + 1))
        assert np.array_equal(out[start(u):start(u + 1)].cpu().numpy().astype(np.int32), want), u
    a, b = start(1000) + 5, start(1100) + 7
    part = dv.all_pairs_scores(a, b, dtype=torch.int8)
    assert torch.equal(part, out[a:b])
    a, b = start(n // 3) + 100, start(n // 3 + 3000) + 7
    part = dv.all_pairs_scores(a, b, dtype=torch.int16)
    assert torch.equal(part, out[a:b].to(torch.int16))


@pytest.mark.parametrize("name", list(SCORINGS))
@pytest.mark.parametrize("n,lmax", [(2304, 13), (2305, 48), (2305, 13), (3073, 36), (6145, 25), (6145, 48)])
def test_triangle_bits_small_windows(name, n, lmax):
    """Blocks of 256 words with windows of 256, 512 and 1024, and the line below
    which three planes stay with the packed kernels: ranges at every byte
    alignment against the oracle (the whole triangle up to 2,305 words)."""
    nw, torch = _nw()
    v = _words(n, SCORINGS[name][0], lmax, seed=7)
    dv, sim, gap = _load(name, v)
    start = lambda u: u * (2 * n - u - 1) // 2
    ranges = [(start(u) + c, start(u + 1)) for u, c in
              [(0, 0), (255, 0), (256, 0), (511, 700), (1023, 0), (1024, 1), (n - 1025, 3), (n - 258, 0), (n - 2, 0)]]
    ranges += [(start(250) + 9, start(262) + 1300), (start(n - 300) + 5, start(n - 200))]
    if n <= 2305:
        ranges.append((0, n * (n - 1) // 2))
    whole = dv.all_pairs_scores(dtype=torch.int16)
    for q, (a, b) in enumerate(ranges):
        buf = torch.full(((b - a) * 2 + 16,), 0x55, dtype=torch.uint8, device="cuda:0")
        rc = nw._lib.nw_all_pairs_scores(dv._h, a, b, 2, ctypes.c_void_p(buf.data_ptr() + q % 4),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == nw.NW_OK
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        got = host[q % 4:q % 4 + (b - a) * 2].copy().view(np.int16)
        want = oracle.triangle(v.symbols, v.offsets, sim, gap, a, b)
        assert np.array_equal(got.astype(np.int32), want), (a, b)
        assert np.array_equal(whole[a:b].cpu().numpy(), got), (a, b)
        assert (host[:q % 4] == 0x55).all() and (host[q % 4 + (b - a) * 2:] == 0x55).all(), (a, b)


@pytest.mark.parametrize("name", list(SCORINGS))
@pytest.mark.parametrize("n,lmax", [(333, 48), (530, 11)])
def test_edges_bits(name, n, lmax):
    """Raw and normalised slices, counting alone, a capacity below the count, ranges and a dense slice."""
    _, torch = _nw()
    v = _words(n, SCORINGS[name][0], lmax, seed=8)
    dv, sim, gap = _load(name, v)
    pairs = n * (n - 1) // 2
    lo, hi = dv.bounds
    slices = [(hi // 2, hi, False, 1), (lo, hi, False, 1), (hi + 1, hi + 5, False, 1), (60, 100, True, 1), (200, 400, True, 3),
              (-350, -10, True, 2), (-1000000, 1000000, True, 1)]
    for q, (a, b, norm, den) in enumerate(slices):
        for i0, i1 in ([(0, pairs)] if q else [(0, pairs), (pairs // 3 + 1, pairs // 2 + 7), (5, 6)]):
            ei, ej, es = oracle.edges(v.symbols, v.offsets, sim, gap, a, b, normalised=norm, den=den, idx_begin=i0, idx_end=i1)[:3]
            i, j, s, count = dv.all_pairs_edges(a, b, normalised=norm, den=den, idx_begin=i0, idx_end=i1)
            assert count == len(ei)
            got = sorted(zip(i.tolist(), j.tolist(), s.tolist()))
            assert got == sorted(zip(map(int, ei), map(int, ej), map(int, es)))
            if count > 10:
                i, j, s, count2 = dv.all_pairs_edges(a, b, normalised=norm, den=den, idx_begin=i0, idx_end=i1, cap=count - 7)
                assert count2 == count and set(zip(i.tolist(), j.tolist(), s.tolist())) <= set(got)


# name -> (generator args of test_gpu_prepass.make_vocab, k): from the size on at
# which the bit-plane pre-pass applies; ties, empty words, odd probe counts
PREPASS = {
    "zipf_131073": (("zipf", 131073, 21), 32),
    "zipf_140003": (("zipf", 140003, 22), 1),
    "uni4_150001": (("uniform", 150001, 23, 4, 0, 12), 63),
    "uni2_132000": (("uniform", 132000, 24, 2, 1, 9), 16),
}

PREPASS_CHILD = r"""
import sys
sys.path.insert(0, sys.argv[1]); sys.path.insert(0, sys.argv[1] + "/tests")
import numpy as np
import test_gpu_bits as T
for name in T.PREPASS:
    np.savez(f"{sys.argv[2]}/{name}.npz", **T.prepass_case(name))
    print("child done", name, flush=True)
"""


def prepass_case(name):
    nw, torch = _nw()
    from test_gpu_prepass import make_vocab
    gen, k = PREPASS[name]
    v = make_vocab(gen)
    alphabet = 40 if gen[0] == "zipf" else gen[3]
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(alphabet, 1, -1, -1))
    ws = torch.zeros(dv.topk_workspace_bytes(k), dtype=torch.uint8, device="cuda")
    s, i, _ = dv.all_pairs_topk(k, hist=False, ws=ws)
    torch.cuda.synchronize()
    o = (8 * v.n + 255) // 256 * 256
    a = ws[:o + 4 * v.n].cpu().numpy()
    return dict(thr=a[:8 * v.n].view(np.uint64).copy(), cnt=a[o:].view(np.uint32).copy(), s=s.cpu().numpy(), i=i.cpu().numpy())


def test_prepass_bits_matches_packed(tmp_path):
    """The bit-plane pre-pass leaves the thresholds, candidate counts and lists of the packed selection."""
    _nw()
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, NW_PREPASS="packed")
    r = subprocess.run([sys.executable, "-c", PREPASS_CHILD, root, str(tmp_path)], env=env, capture_output=True, text=True,
                       timeout=110)
    assert r.returncode == 0, r.stdout + r.stderr
    for name in PREPASS:
        got, want = prepass_case(name), np.load(tmp_path / f"{name}.npz")
        for key in ("thr", "cnt", "s", "i"):
            assert np.array_equal(got[key], want[key]), (name, key, int((got[key] != want[key]).sum()))


@pytest.mark.parametrize("name,n,lmax,k", [
    ("plain", 16384, 12, 3), ("plain", 16385, 12, 3), ("plain", 5000, 12, 2), ("levenshtein", 5000, 9, 63),
    ("levenshtein", 17000, 9, 16), ("matrix_64", 17000, 14, 1), ("weight_8", 3000, 20, 8)])
def test_topk_phases(name, n, lmax, k):
    """Both sides of the rule for one main-pass phase: sampled rows and the whole histogram's count."""
    _, torch = _nw()
    v = _words(n, SCORINGS[name][0], lmax, seed=11)
    dv, sim, gap = _load(name, v)
    sc, ix, h = dv.all_pairs_topk(k)
    torch.cuda.synchronize()
    assert int(h.sum()) == n * (n - 1) // 2
    for r0 in (0, 255, n // 2, n - 40):
        r1 = min(n, r0 + 40)
        ws, wi, _ = oracle.topk_rows(v.symbols, v.offsets, sim, gap, k, r0=r0, r1=r1)
        assert np.array_equal(sc.cpu().numpy()[r0:r1].astype(np.int32), ws)
        assert np.array_equal(ix.cpu().numpy()[r0:r1], wi)
