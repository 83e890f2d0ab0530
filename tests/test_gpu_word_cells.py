"""Batches on the 16-bit kernel whose cells are added as 32-bit words, and those just outside its rule: letters' scores at both
ends of a byte, values at the top of 15 bits, two to five letters, invalid letters, empty sides, both gap kinds, with and without
CIGARs: all equal to the oracle's."""
import numpy as np
import pytest

import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _batch(seed, mode, alphabet, go, ge, match, mismatch, traceback, top=256, n_pairs=100003):
    """Mostly tiny pairs (so many that the batch runs one pair per lane), a few of up to top letters, some of them related."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 13, (n_pairs, 2))
    big = rng.choice(n_pairs, 60, replace=False)
    lens[big] = rng.integers(top - 20, top + 1, (60, 2))
    lens[big[0]] = (top, top)
    lens[big[1:4]] = [(top, 1), (1, top), (0, top)]
    qo = np.concatenate([[0], np.cumsum(lens[:, 0])]).astype(np.int64)
    so = np.concatenate([[0], np.cumsum(lens[:, 1])]).astype(np.int64)
    q = rng.integers(0, alphabet, int(qo[-1]), dtype=np.uint8)
    s = rng.integers(0, alphabet, int(so[-1]), dtype=np.uint8)
    for p in np.concatenate([big[0:1], big[4::3]]):
        k = min(lens[p])
        s[so[p]:so[p] + k] = q[qo[p]:qo[p] + k]
        if p != big[0]:
            s[so[p] + k // 2] = (s[so[p] + k // 2] + 1) % alphabet
    return synth.Workload("word", mode, alphabet, go, ge, q, qo, s, so, match=match, mismatch=mismatch, traceback=traceback)


def _check(w, traceback):
    import paper_2002_04561_amd as aln
    gres, gcig = run_gpu(w, aln.TRACEBACK if traceback else aln.SCORE_ONLY)
    ores, ocig = run_oracle(w, traceback)
    bad = compare(w, gres, gcig, ores, ocig, "word")
    assert not bad, bad[:3]


@pytest.mark.parametrize("mode", [0, 2], ids=["global", "semi"])
@pytest.mark.parametrize("traceback", [False, True], ids=["score", "cigar"])
@pytest.mark.parametrize("alphabet,go,ge,match,mismatch", [
    (4, -5, -2, 1, -4), (4, 0, -1, 2, -2), (4, 0, -1, 2, -3), (4, -3, -1, 2, -5), (4, -3, -1, 2, -6),
    (4, -40, -20, 43, -20), (4, -10, -20, 43, -20), (4, 0, -20, 44, -20), (4, -100, -1, 100, 10), (4, -100, -2, 100, -100),
    (4, -124, -2, 127, -100), (4, -125, -2, 127, -100), (2, -3, -1, 2, -3), (3, -3, -1, -1, -2), (5, -3, -1, 2, -3)])
def test_word_cells(gpu, mode, traceback, alphabet, go, ge, match, mismatch):
    w = _batch(alphabet - go + match, mode, alphabet, go, ge, match, mismatch, traceback, top=100 if match >= 100 else 256)
    _check(w, traceback)


@pytest.mark.parametrize("mode", [0, 2], ids=["global", "semi"])
@pytest.mark.parametrize("alphabet", [2, 4])
def test_invalid_letters(gpu, mode, alphabet):
    w = _batch(5, mode, alphabet, -3, -1, 2, -3, True, top=70, n_pairs=40000)
    rng = np.random.default_rng(6)
    w.q[rng.integers(0, len(w.q), 50)] = alphabet
    w.s[rng.integers(0, len(w.s), 50)] = 255
    import paper_2002_04561_amd as aln
    gres, gcig = run_gpu(w, aln.TRACEBACK)
    bad = np.array([bool((w.q[w.q_off[p]:w.q_off[p + 1]] >= alphabet).any() or (w.s[w.s_off[p]:w.s_off[p + 1]] >= alphabet).any())
                    for p in range(len(w.q_off) - 1)])
    assert (((gres["flags"] & aln.RES_BAD_CODE) != 0) == bad).all()
    assert not np.any(gres["score"][bad])
    w.q[w.q >= alphabet] = 0
    w.s[w.s >= alphabet] = 0
    ores, ocig = run_oracle(w, True)
    for k in ("score", "q_begin", "q_end", "s_begin", "s_end", "cigar_len"):
        assert (gres[k][~bad] == ores[k][~bad]).all(), k
    assert [c for c, b in zip(gcig, bad) if not b] == [c for c, b in zip(ocig, bad) if not b]
