"""Band wavefronts whose scores sigma - 2 ge leave a signed byte: the bytes are kept lowered by what the largest of them exceeds
127, and a cell adds that back.  Schemes on either side of each limit (the largest score at 127 and 128, the spread at 254 and
255 byte values, the largest score at 126 and 127 where a pad letter would become a match, the offset at 127 and 128 over more
than four letters), in every mode, with both gap models, with and without CIGARs: equal to the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# alphabet, match, mismatch, gap extend
SCHEMES = {
    "largest_127": (4, 107, -20, -10), "largest_128": (4, 108, -20, -10), "dna_match_91": (4, 91, -114, -30),
    "spread_254": (4, 126, -128 + 1, -64), "spread_255": (4, 126, -127, -65), "pads_mismatch": (4, 126, -100, -200),
    "pads_match": (4, 127, -100, -200), "two_letters": (2, 5, -4, -70), "extend_200": (3, 5, -4, -200),
    "lanes_offset_127": (5, 54, -60, -100), "lanes_offset_128": (5, 55, -60, -100), "lanes_20": (20, 11, -4, -70),
}


def _pairs(seed, alphabet):
    rng = np.random.default_rng(seed)
    qs, ss = [], []
    for n, m in [(1, 1), (1, 300), (300, 1), (3, 5), (63, 66), (64, 64), (65, 31), (255, 257), (256, 256), (257, 255), (511, 90),
                 (90, 511), (700, 701), (1030, 640)]:
        a = rng.integers(0, alphabet, n, dtype=np.uint8)
        b = rng.integers(0, alphabet, m, dtype=np.uint8)
        k = min(n, m) // 2
        b[m - k:] = a[n - k:]  # ends that match, beside the pad columns
        qs += [a, a[::-1].copy()]
        ss += [b, b[::-1].copy()]
    return qs, ss


def _workload(mode, scheme, go, seed):
    alphabet, match, mismatch, ge = SCHEMES[scheme]
    q, qo = synth.pack(_pairs(seed, alphabet)[0])
    s, so = synth.pack(_pairs(seed, alphabet)[1])
    return synth.Workload("large_scores", mode, alphabet, go, ge, q, qo, s, so, match=match, mismatch=mismatch, traceback=True)


MODES = pytest.mark.parametrize("mode", [synth.GLOBAL, synth.LOCAL, synth.SEMIGLOBAL], ids=["global", "local", "semiglobal"])


@pytest.mark.parametrize("go", [0, -400], ids=["linear", "affine"])
@pytest.mark.parametrize("scheme", list(SCHEMES))
@MODES
def test_batches(gpu, mode, scheme, go):
    import paper_2002_04561_amd as aln
    w = _workload(mode, scheme, go, 80)
    scores, traced = run_oracle(w, False), run_oracle(w, True)
    for group in (1, 4):
        config = aln.BatchConfig(wf_min_cells=1, wf_group=group)
        gres, _ = run_gpu(w, aln.SCORE_ONLY, config=config)
        bad = compare(w, gres, None, scores[0], None, "scores")
        assert not bad, (group, bad[:3])
    bad = compare(w, *run_gpu(w, aln.TRACEBACK, config=aln.BatchConfig(wf_min_cells=1)), *traced, "cigars")
    assert not bad, bad[:3]


@pytest.mark.parametrize("go", [0, -400], ids=["linear", "affine"])
@pytest.mark.parametrize("scheme", ["dna_match_91", "pads_mismatch", "pads_match", "lanes_20"])
@MODES
def test_one_pair_in_linear_space(gpu, mode, scheme, go):
    import torch

    import paper_2002_04561_amd as aln
    alphabet, match, mismatch, ge = SCHEMES[scheme]
    rng = np.random.default_rng(81)
    q = rng.integers(0, alphabet, 2300, dtype=np.uint8)
    s = np.concatenate([rng.integers(0, alphabet, 700, dtype=np.uint8), q[200:1400], q[1450:2250],
                        rng.integers(0, alphabet, 333, dtype=np.uint8)])
    la = aln.LongAligner(aln.Scoring(mode, alphabet, go, ge, match=match, mismatch=mismatch), torch.from_numpy(q).cuda(),
                         torch.from_numpy(s).cuda(), aln.TRACEBACK | aln.LINEAR_SPACE)
    la.run()
    torch.cuda.synchronize()
    g = la.result()
    r = oracle.align(oracle.Scoring.simple(mode, alphabet, match, mismatch, go, ge), q, s, traceback=True, impl="checkpointed")
    got = tuple(int(g[f]) for f in ("score", "q_begin", "q_end", "s_begin", "s_end", "flags")) + (la.cigar_runs(),)
    assert got == (r.score, r.q_begin, r.q_end, r.s_begin, r.s_end, 0, r.cigar)
