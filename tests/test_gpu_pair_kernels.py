"""Traceback batches on both sides of the rule that runs short batches one pair per wave and long ones one pair per lane:
tiny pairs, 257-row pairs, empty sides, invalid letters and 32-bit redo flags, in all modes, each equal to the oracle; and
aln_traceback with forward results whose end cells, scores or letters do not fit."""
import numpy as np
import pytest

import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _batch(seed, n_pairs, top, mode, go=-3, ge=-1, alphabet=4, subst=None):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, top + 1, (n_pairs, 2))
    lens[0] = (top, top)
    q_off = np.concatenate([[0], np.cumsum(lens[:, 0])]).astype(np.int64)
    s_off = np.concatenate([[0], np.cumsum(lens[:, 1])]).astype(np.int64)
    q = rng.integers(0, alphabet, int(q_off[-1]), dtype=np.uint8)
    s = rng.integers(0, alphabet, int(s_off[-1]), dtype=np.uint8)
    kw = dict(match=2, mismatch=-3) if subst is None else dict(subst=subst)
    return synth.Workload("pairs", mode, alphabet, go, ge, q, q_off, s, s_off, traceback=True, **kw)


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
@pytest.mark.parametrize("n_pairs,top", [(1, 3), (130, 70), (60, 300), (12, 1024), (70001, 12)])
@pytest.mark.parametrize("bits", [16, 32])
def test_short_and_long_batches(gpu, mode, go, n_pairs, top, bits):
    import paper_2002_04561_amd as aln
    w = _batch(n_pairs + mode, n_pairs, top, mode, go)
    flags = aln.TRACEBACK | (aln.FORCE_INT32 if bits == 32 else 0)
    gres, gcig = run_gpu(w, flags)
    ores, ocig = run_oracle(w, True)
    bad = compare(w, gres, gcig, ores, ocig, "pairs")
    assert not bad, bad[:3]
    assert not np.any(gres["flags"])


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
def test_protein_and_redo_flags(gpu, mode):
    """The 20-letter profile; and with gaps of -30 a letter, pairs whose 16-bit range is not provable carry the redo flag of
    the 16-bit path whichever kernel runs them (one per wave here, one per lane in the long batch)."""
    import paper_2002_04561_amd as aln
    sig = synth.protein_sigma(np.random.default_rng(1))
    w = _batch(3, 50, 400, mode, -11, -1, 20, sig)
    bad = compare(w, *run_gpu(w, aln.TRACEBACK), *run_oracle(w, True), "protein")
    assert not bad, bad[:3]
    n = 510  # 2^18 cells and more run on the band wavefront
    a = np.random.default_rng(2).integers(0, 4, n, dtype=np.uint8)
    q, qo = synth.pack([a, a[:40]])
    s, so = synth.pack([a, a[:50]])
    w = synth.Workload("redo", mode, 4, -3, -30, q, qo, s, so, match=100, mismatch=-3, traceback=True)
    gres, gcig = run_gpu(w, aln.TRACEBACK)
    assert gres["flags"].tolist() == [aln.RES_INT32_REDO, 0]
    ores, ocig = run_oracle(w, True)
    assert [int(x) for x in gres["score"]] == [int(x) for x in ores["score"]] and gcig == ocig


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
def test_bad_letters_and_ends(gpu, mode):
    """Both kernels give the same flags: invalid letters in a query, in a subject, beside an empty side and past the end cell, an
    end cell outside the matrix, and a score that is not H there (an invalid letter is on no alignment, so it decides that
    too).  7 pairs run one per wave, 10,500 one per lane."""
    import torch

    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(7)
    qs = [rng.integers(0, 4, k, dtype=np.uint8) for k in (30, 30, 30, 0, 30, 30, 30)]
    ss = [rng.integers(0, 4, k, dtype=np.uint8) for k in (33, 33, 33, 20, 33, 33, 33)]
    qs[1][5] = 9
    ss[2][32] = 4
    ss[3][3] = 4
    got = []
    for copies in (1, 1500):
        w = synth.Workload("bad", mode, 4, -3, -1, *synth.pack(qs * copies), *synth.pack(ss * copies), match=2, mismatch=-3,
                           traceback=True)
        gres, _ = run_gpu(w, aln.TRACEBACK)
        assert gres["flags"].tolist() == [0, 4, 4, 4, 0, 0, 0] * copies
        assert not np.any(gres["score"].reshape(copies, 7)[:, 1:4]) and not np.any(gres["cigar_len"].reshape(copies, 7)[:, 1:4])
        # aln_traceback from end cells that a scoring over 10 letters found, where 4 and 9 are valid, and spoilt ones
        good, _ = run_gpu(synth.Workload("good", mode, 10, -3, -1, w.q, w.q_off, w.s, w.s_off, match=2, mismatch=-3), 0)
        fwd = np.ascontiguousarray(good)
        fwd["s_end"][4::7] = 34
        fwd["score"][5::7] += 1
        fwd["flags"][6::7] = aln.RES_TOO_LONG
        q, qo, s, so = aln.to_device(w)
        dev = torch.from_numpy(fwd.view(np.int32).copy()).cuda()
        sc = aln.Scoring(mode, 4, -3, -1, match=2, mismatch=-3)
        res, runs = aln.traceback_pairs(sc, q, qo, s, so, 30, 33, dev)
        assert res["flags"][[0, 4, 5, 6]].tolist() == [0, aln.RES_BAD_END, aln.RES_BAD_END, aln.RES_TOO_LONG]
        got.append([(res[k].tolist(), runs[k]) for k in range(7 * copies)])
    assert got[1] == got[0] * 1500
