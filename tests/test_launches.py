"""What the calls launch, on the CPU: a preloaded HIP runtime (hip_recorder.c)
records kernels, grids and streams and runs nothing, so the host's rules -- which
kernel a dictionary takes, how a launch is cut, on which stream it goes -- are
tested where there is no GPU.  Every check runs in one child process per group.
"""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests")


class _Record(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 512), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3),
                ("lds", ctypes.c_uint64), ("stream", ctypes.c_uint64)]


class Recorder:
    """The recorder and libnw in this (child) process."""

    def __init__(self):
        import paper_2509_01654_amd as nw
        self.nw, self.lib = nw, nw.load_library()
        self.hip = ctypes.CDLL(None)
        self.hip.rec_get.restype = ctypes.POINTER(_Record)
        self.P = ctypes.c_void_p

    def load(self, symbols, offsets, sc):
        symbols = np.ascontiguousarray(symbols, dtype=np.uint8)
        offsets = np.ascontiguousarray(offsets, dtype=np.uint64)
        h = ctypes.c_void_p()
        c = sc._c()
        rc = self.lib.nw_load_vocab(symbols.ctypes.data, offsets.ctypes.data, offsets.shape[0] - 1, ctypes.byref(c),
                                    self.P(1 << 40), 1 << 40, None, ctypes.byref(h))
        assert rc == 0, self.lib.nw_last_error()
        return h

    def launches(self, fn, *args):
        """[(kernel, grid, threads, lds, stream)] of one call."""
        self.hip.rec_clear()
        rc = fn(*args)
        assert rc == 0, self.lib.nw_last_error()
        out = []
        for i in range(self.hip.rec_count()):
            r = self.hip.rec_get(i).contents
            out.append((r.name.decode(), tuple(r.grid), r.block[0], r.lds, r.stream))
        return out


def words(n, alphabet, lo, hi, seed=5):
    rng = np.random.default_rng(seed)
    lengths = rng.integers(lo, hi + 1, size=n)
    offsets = np.zeros(n + 1, np.uint64)
    np.cumsum(lengths, out=offsets[1:])
    return rng.integers(0, alphabet, size=int(lengths.sum())), offsets


@pytest.fixture(scope="module")
def recorder_library(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_recorder.c"), "-ldl"], check=True)
    return so


def _child(recorder_library, check):
    """Run check_<name>(Recorder) in a child with the recorder preloaded."""
    env = dict(os.environ)
    env["LD_PRELOAD"] = recorder_library + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {HERE!r}]\n"
            f"import test_launches as T\nT.{check}(T.Recorder())\nprint('checked')\n")
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "checked" in r.stdout, r.stdout[-3000:] + r.stderr[-3000:]


def _topk_bytes(R, h, k):
    out = ctypes.c_uint64()
    assert R.lib.nw_topk_workspace_bytes(h, k, ctypes.byref(out)) == 0
    return out.value


def check_packed_topk(R):
    # 17,000 words, one of eight a probe: about 8 (k + 1) candidates of a word,
    # twice that as its list (a sixteenth: 16 (k + 1))
    n, k = 17000, 63
    h = R.load(*words(n, 40, 0, 12), R.nw.Scoring(40, 4, -1, -2))
    need = _topk_bytes(R, h, k)
    assert need < 8 * n * (2.5 * 8 * (k + 1))
    # and no first phase of its own: too few words would get a closer threshold
    P = R.P
    for k in (16, 63):
        names = [x[0] for x in R.launches(R.lib.nw_all_pairs_topk_async, h, k, P(1 << 41), P(1 << 42), None, P(1 << 43),
                                          _topk_bytes(R, h, k), None)]
        assert any("k_topk_code" in x for x in names) and not any("tighten" in x for x in names), names


def test_packed_topk_thresholds(recorder_library):
    """The packed main pass pays more for a candidate than the plane kernels do."""
    _child(recorder_library, "check_packed_topk")


def _edges(R, h, a, b):
    f = R.nw._EdgeFilter(1, 60, 100, 1)
    P = R.P
    return R.launches(R.lib.nw_all_pairs_edges, h, a, b, ctypes.byref(f), P(1 << 41), P(1 << 42), P(1 << 43), 1 << 20,
                      P(1 << 44), None)


def check_few_lengths_edges(R):
    # 2,300 words of one length: 45 tiles of eight row groups, one workgroup a tile before
    for n, length, want in ((2300, 24, 300), (700, 48, 40)):
        for sc in (R.nw.Scoring(40, 1, -1, -1), R.nw.Scoring(40, 0, -1, -1)):
            h = R.load(*words(n, 40, length, length), sc)
            grids = [g for name, g, *_ in _edges(R, h, 0, n * (n - 1) // 2) if "k_edges_bits" in name]
            assert sum(x * y * z for x, y, z in grids) >= want, grids


def test_edges_of_few_lengths_fill_the_chip(recorder_library):
    _child(recorder_library, "check_few_lengths_edges")


def check_tiny_edges(R):
    for sc, least in ((R.nw.Scoring(40, 1, -1, -1), 8), (R.nw.Scoring(40, 0, -1, -1), 32)):
        for n, planes in ((2, False), (least - 1, False), (least, True)):
            h = R.load(*words(n, 40, 48, 48), sc)
            names = [x[0] for x in _edges(R, h, 0, n * (n - 1) // 2)]
            assert any("k_edges_bits" in x for x in names) == planes, (n, names)


def test_edges_of_a_few_words_stay_packed(recorder_library):
    _child(recorder_library, "check_tiny_edges")


def _triangle(R, h, a, b, dtype=2):
    return R.launches(R.lib.nw_all_pairs_scores, h, a, b, dtype, R.P(1 << 41), None)


def _planes(launches):
    kinds = {"k_tri_bits" in x[0] for x in launches}
    assert len(kinds) == 1, launches
    return kinds.pop()


PLAIN, MATRIX = (1, -1, -1), (0, -1, -1)   # two planes; three


def check_triangle_routes(R):
    # scoring, words, lengths, share of the triangle, planes or not: calls where one
    # side was measured well ahead
    for sc, n, lo, hi, share, planes in [
            (PLAIN, 2, 12, 12, 1, False), (PLAIN, 4, 48, 48, 1, False), (PLAIN, 300, 1, 16, 1, True),
            (PLAIN, 200, 24, 24, 1, False), (PLAIN, 700, 48, 48, 1, False), (PLAIN, 1500, 24, 24, 1, True),
            (PLAIN, 2000, 1, 20, 1, True), (PLAIN, 300, 22, 26, 1, False), (PLAIN, 1500, 44, 48, 1, True),
            (PLAIN, 5000, 1, 48, 1e-4, True), (MATRIX, 700, 12, 12, 1, False), (MATRIX, 3100, 12, 12, 1, True),
            (MATRIX, 300, 1, 12, 1, True), (MATRIX, 2304, 1, 16, 1, False), (MATRIX, 6000, 1, 13, 1, True),
            (MATRIX, 5000, 30, 48, 0.01, False), (MATRIX, 16000, 30, 48, 1e-5, True), (MATRIX, 12000, 30, 48, 0.1, True),
            (MATRIX, 17000, 1, 48, 1e-4, True)]:
        h = R.load(*words(n, 40, lo, hi), R.nw.Scoring(40, *sc))
        pairs = n * (n - 1) // 2
        a = pairs // 3 if share < 1 else 0
        got = _planes(_triangle(R, h, a, min(pairs, a + max(1, int(pairs * share)))))
        assert got == planes, (sc, n, lo, hi, share, got)


def test_small_triangles_stay_packed(recorder_library):
    """Dictionaries of a few words or few lengths, and ranges of few pairs under three planes."""
    _child(recorder_library, "check_triangle_routes")


def check_few_lengths_triangle(R):
    for sc, n, length in ((PLAIN, 2300, 24), (MATRIX, 4000, 24)):
        h = R.load(*words(n, 40, length, length), R.nw.Scoring(40, *sc))
        out = _triangle(R, h, 0, n * (n - 1) // 2)
        assert _planes(out) and sum(x * y * z for _, (x, y, z), *_ in out) >= 500, out


def test_triangle_of_few_lengths_fills_the_chip(recorder_library):
    _child(recorder_library, "check_few_lengths_triangle")


def check_column_layout(R):
    # nw::launch_column_layout(vocab, lengths, columns, window, slots, out, stream)
    fn = R.lib._ZN2nw20launch_column_layoutERKNS_8DevVocabEPKhPKtilPjP12ihipStream_t
    fn.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    fn.restype = ctypes.c_int
    vocab = ctypes.create_string_buffer(4096)
    for slots in (256, 3072 * 1000, 400_000_128, 2_147_480_576):
        R.hip.rec_clear()
        assert fn(vocab, None, None, 1024, slots, R.P(1 << 41), None) == 0, slots
        threads = sum(r.grid[0] * r.block[0] for r in (R.hip.rec_get(i).contents for i in range(R.hip.rec_count())))
        assert 12 * slots <= threads < 12 * slots + 256 * R.hip.rec_count(), (slots, threads)


def test_column_layout_of_the_largest_dictionaries(recorder_library):
    """A grid holds fewer than 2^32 threads: the layout of 357 million words and more goes in several launches."""
    _child(recorder_library, "check_column_layout")


def check_query_stream(R):
    h = R.load(*words(20000, 40, 1, 32), R.nw.Scoring(40, 1, -1, -1))
    P, stream = R.P, 0x7770
    for n in (1, 2, 64, 300, 1000):   # the largest goes up by a copy, the others as kernel arguments
        qs, qo = words(n, 40, 0, 40, seed=n)
        qs = np.ascontiguousarray(qs, dtype=np.uint8)
        out = R.launches(R.lib.nw_query, h, qs.ctypes.data, qo.ctypes.data, n, 16, P(1 << 41), P(1 << 42), P(1 << 43),
                         1 << 40, P(stream))
        assert any("k_query" in x[0] for x in out)
        assert {x[4] for x in out} == {stream}, (n, out)
        assert sum(x[1][0] for x in out if "k_query" in x[0]) >= (n + 1) // 2   # every row pair


def test_queries_run_on_the_callers_stream(recorder_library):
    """A query waits for no other caller's work: nothing of it goes to the library's streams."""
    _child(recorder_library, "check_query_stream")


def check_load(R):
    for sc, lmax, planes in ((PLAIN, 20, True), (MATRIX, 20, True), ((4, -1, -2), 20, False), (PLAIN, 49, False)):
        R.hip.rec_clear()
        R.load(*words(3000, 40, lmax, lmax), R.nw.Scoring(40, *sc))
        names = [R.hip.rec_get(i).contents.name.decode() for i in range(R.hip.rec_count())]
        assert any("k_column_layout" in x for x in names) == planes, (sc, lmax, names)


def test_load_lays_out_planes_only_where_they_run(recorder_library):
    _child(recorder_library, "check_load")


def _autotune(R, scoring, cache):
    hs = [R.load(*words(n, 20, 0, lmax, seed=n), R.nw.Scoring(20, *scoring)) for n, lmax in ((300, 10), (900, 16))]
    vh = (ctypes.c_void_p * 2)(*[h.value for h in hs])
    oh = (ctypes.c_void_p * 2)(1 << 41, 1 << 42)
    best, ms = R.nw._BatchOptions(), ctypes.c_float()
    rc = R.lib.nw_batch_autotune(vh, 2, oh, R.nw.NW_I16, R.P(1 << 43), 1 << 40, None, cache.encode(), ctypes.byref(best),
                                 ctypes.byref(ms))
    assert rc == 0, R.lib.nw_last_error()
    for h in hs:
        R.lib.nw_free_vocab(h)
    return open(cache).read().splitlines(), best, ms.value


def check_autotune(R):
    import tempfile
    # (the recorder has no graphs: a candidate that captured one would fail here)
    with tempfile.TemporaryDirectory() as d:
        cache = d + "/tune.jsonl"
        for n, sc in enumerate([PLAIN, MATRIX, (4, -1, -2), (8, -1, -2)]):
            lines, first, _ = _autotune(R, sc, cache)
            assert len(lines) == n + 1, "another scoring's line answered"
            lines, again, _ = _autotune(R, sc, cache)
            assert len(lines) == n + 1, "its own line did not"
            assert bytes(first) == bytes(again) and first.use_graph == (first.class_width != 0)
        # a line without the kernels' generation and the scorings, as it was written before
        old = d + "/old.jsonl"
        with open(old, "w") as f:
            lens = [np.diff(words(n, 20, 0, lmax, seed=n)[1].astype(np.int64)) for n, lmax in ((300, 10), (900, 16))]
            key = "recorder/|dt2" + "".join(f"|{l.size}:{l.max()}:20:{l.sum()}" for l in lens)
            f.write('{"key": "%s", "class_width": 1, "wg_per_cu": 2, "pairs_per_item": 16, "use_graph": 1, "ms": 0.001}\n' % key)
        lines, best, ms = _autotune(R, PLAIN, old)
        assert len(lines) == 2 and ms > 0.5, "a line of earlier kernels answered"


def test_autotune_cache_tells_scorings_and_kernels_apart(recorder_library):
    _child(recorder_library, "check_autotune")


def check_packed_routes(R):
    # the scorings of the GPU tests of the packed kernels do take them
    h = R.load(*words(17000, 40, 0, 20), R.nw.Scoring(40, 4, -1, -2))
    n, P = 17000, R.P
    tri = {x[0] for x in _triangle(R, h, 0, n * (n - 1) // 2)}
    assert all("k_tri_code" in x for x in tri) and any("Li1E" in x for x in tri) and any("Li2E" in x for x in tri), tri
    assert all("k_edges_tiled" in x[0] for x in _edges(R, h, 0, 5000) if "k_edges" in x[0])
    top = [x[0] for x in R.launches(R.lib.nw_all_pairs_topk_async, h, 16, P(1 << 41), P(1 << 42), P(1 << 44), P(1 << 43),
                                    _topk_bytes(R, h, 16), None)]
    assert any("k_topk_code" in x for x in top) and not any("bits" in x for x in top), top


def test_packed_scorings_take_the_packed_kernels(recorder_library):
    _child(recorder_library, "check_packed_routes")
