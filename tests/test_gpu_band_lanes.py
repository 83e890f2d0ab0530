"""The band wavefront's two kinds of lanes: values held as floats while every one fits 2^23 consecutive integers, and
integers beyond.  Pairs just inside and just outside that range (min(n, m) max(sigma, 0) + (n + m + 512) |ge| against
2^23 - 2^20, which large gap extensions reach), in all modes, with byte profiles and with the 32-bit table, one pair
and batches, scores and CIGARs: all equal to the oracle's."""
import numpy as np
import pytest

import synth
from helpers import compare, oracle_scoring, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _pair(seed, n, m):
    """A subject with mutated copies of the query in it, so that local and semi-global optima are not trivial."""
    rng = np.random.default_rng(seed)
    a = rng.integers(0, 4, n, dtype=np.uint8)
    b = rng.integers(0, 4, m, dtype=np.uint8)
    for at in (m // 3, m - n - 5):
        c = synth.mutate_geometric(rng, a, 0.05, 0.005, 2.0)[:n]
        b[max(at, 0):max(at, 0) + len(c)] = c[:max(0, m - max(at, 0))]
    return a, b


def _check_long(w, flags):
    import torch

    import oracle
    import paper_2002_04561_amd as aln
    a, b = w.pair(0)
    q, s = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    la = aln.LongAligner(aln.scoring_of(w), q, s, flags)
    la.run()
    torch.cuda.synchronize()
    g = la.result()
    tb = bool(flags & aln.TRACEBACK)
    r = oracle.align(oracle_scoring(w), a, b, traceback=tb, impl="affine" if tb else "linspace")
    assert (int(g["score"]), int(g["q_end"]), int(g["s_end"]), int(g["flags"])) == (r.score, r.q_end, r.s_end, 0)
    if tb:
        assert (int(g["q_begin"]), int(g["s_begin"]), la.cigar_runs()) == (r.q_begin, r.s_begin, r.cigar)


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("m", [118000, 125000], ids=["float_lanes", "integer_lanes"])
def test_byte_profiles(gpu, mode, m):
    """|ge| = 60 keeps sigma - 2 ge in a byte; 300 x 118000 fits float lanes, 300 x 125000 does not."""
    import paper_2002_04561_amd as aln
    a, b = _pair(5, 300, m)
    q, qo = synth.pack([a])
    s, so = synth.pack([b])
    w = synth.Workload("lanes", mode, 4, -20, -60, q, qo, s, so, match=5, mismatch=-4)
    _check_long(w, aln.SCORE_ONLY)


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("ge", [-6000, -14000], ids=["float_lanes", "integer_lanes"])
def test_table_profiles(gpu, mode, ge):
    """Large gap scores take the 32-bit table: one pair with its CIGAR (codes kept, and in linear space), and a batch
    on bands of their own and in groups."""
    import paper_2002_04561_amd as aln
    a, b = _pair(6, 300, 390)
    q, qo = synth.pack([a])
    s, so = synth.pack([b])
    w = synth.Workload("lanes", mode, 4, -3, ge, q, qo, s, so, match=5, mismatch=-4)
    _check_long(w, aln.SCORE_ONLY)
    _check_long(w, aln.TRACEBACK)
    _check_long(w, aln.TRACEBACK | aln.LINEAR_SPACE)
    pairs = [_pair(20 + k, int(n), int(n) + 40) for k, n in enumerate((1, 63, 64, 255, 256, 257, 330))]
    q, qo = synth.pack([x for x, _ in pairs])
    s, so = synth.pack([y for _, y in pairs])
    w = synth.Workload("lanes", mode, 4, -3, ge, q, qo, s, so, match=5, mismatch=-4)
    ores, _ = run_oracle(w, False)
    for group in (1, 4):
        gres, _ = run_gpu(w, aln.SCORE_ONLY, config=aln.BatchConfig(wf_min_cells=1, wf_group=group))
        bad = compare(w, gres, None, ores, None, "lanes")
        assert not bad, bad[:3]
