"""Top-k thresholds of dictionaries whose order repeats.

The threshold pre-pass looks at a subset of the words.  Dictionaries that
alternate between two kinds of words with a period that divides the subset's
stride must not show it one kind only: the other kind's thresholds would then
be far too low, its candidate lists would overflow and be recomputed one word at
a time.  A few overflows are ordinary; the lists are exact in any case.
"""
import numpy as np
import pytest

import oracle
from synth import vocab_from_words

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _alternating(n, period, seed=4):
    """Every period-th word is long and unlike the rest, which are short and alike."""
    rng = np.random.default_rng(seed)
    return vocab_from_words([rng.integers(0, 40, size=30) if i % period == 0 else
                             rng.integers(0, 6, size=int(rng.integers(5, 9))) for i in range(n)], 40)


@pytest.mark.parametrize("n,period", [(4096, 2), (8192, 4), (8192, 8), (16384, 16), (32768, 16), (140000, 17)])
def test_periodic_dictionary_keeps_its_lists(n, period):
    import paper_2509_01654_amd as nw
    print(f"[gpu case] top-16 of {n} words with period {period}", flush=True)
    v = _alternating(n, period)
    dv = nw.Vocab(v.symbols, v.offsets, nw.Scoring(40, 1, -1, -1))
    k = 16
    s, i, _ = dv.all_pairs_topk(k, hist=False)
    torch.cuda.synchronize()
    assert dv.topk_overflow_words() <= n // 100
    s, i = s.cpu().numpy().astype(np.int32), i.cpu().numpy()
    sim = oracle.sim_matrix(40, 1, -1)
    for r0 in (0, n // 2 + 1, n - 9):
        ws, wi, _ = oracle.topk_rows(v.symbols, v.offsets, sim, -1, k, r0=r0, r1=r0 + 9)
        np.testing.assert_array_equal(i[r0:r0 + 9], wi)
        np.testing.assert_array_equal(s[r0:r0 + 9], ws)
