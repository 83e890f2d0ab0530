"""Tracebacks on the band wavefront (codes stored a cell at a time, walked by one wave a pair) whose walks leave the diagonal or
whose subjects have few letters, where a band's first columns and its last fall into one group of 4 steps: single pairs with
ALN_STORED_CODES, and batches of pairs longer than 1024 on a side, which the planner sends there, with bands in groups and
on their own; and the same scores without CIGARs.  All equal to the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from helpers import compare, oracle_scoring, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# around the walk's windows: 11 columns right and 14 left of the diagonal, rectangles of 32 and 128 columns, 128 and 32 rows
GAPS = (10, 11, 12, 13, 14, 15, 16, 31, 32, 33, 64, 65, 127, 128, 129, 300)


def _gapped(rng, n, gap):
    a, ins = rng.integers(0, 4, n, dtype=np.uint8), rng.integers(0, 4, gap, dtype=np.uint8)
    return a, np.concatenate([a[:n // 2 + 1], ins, a[n // 2 + 1:]])


def _few_columns(rng, n):
    out = []
    for m in (1, 2, 3, 4, 5, 59, 60, 61, 62, 63, 64, 65, 66, 67):
        a = rng.integers(0, 4, n, dtype=np.uint8)
        out.append((a, np.resize(a[n // 2:], m).copy()))
    return out


def _workload(pairs, mode, go):
    q, qo = synth.pack([a for a, _ in pairs])
    s, so = synth.pack([b for _, b in pairs])
    return synth.Workload("walks", mode, 4, go, -1, q, qo, s, so, match=5, mismatch=-4, traceback=True)


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
def test_single_pairs(gpu, mode, go):
    import torch

    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(10 + mode)
    pairs = []
    for gap in GAPS:
        a, b = _gapped(rng, 260, gap)
        pairs += [(a, b), (b, a)]
    pairs += _few_columns(rng, 300) + [(b, a) for a, b in _few_columns(rng, 90)]
    w = _workload(pairs, mode, go)
    for k, (a, b) in enumerate(pairs):
        la = aln.LongAligner(aln.scoring_of(w), torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(),
                             aln.TRACEBACK | aln.STORED_CODES)
        aln.aln_profile_enable(True)
        aln.aln_profile_reset()
        la.run()
        torch.cuda.synchronize()
        ran = aln.aln_profile_read()
        aln.aln_profile_enable(False)
        assert list(ran) == ["wavefront_i32_traceback"], ran
        g, r = la.result(), oracle.align(oracle_scoring(w), a, b, traceback=True)
        got = tuple(int(g[f]) for f in ("score", "q_begin", "q_end", "s_begin", "s_end", "flags")) + (la.cigar_runs(),)
        assert got == (r.score, r.q_begin, r.q_end, r.s_begin, r.s_end, 0, r.cigar), (k, len(a), len(b))


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
@pytest.mark.parametrize("group", [1, 4], ids=["bands_alone", "bands_in_groups"])
def test_batches(gpu, mode, go, group):
    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(20 + mode)
    pairs = []
    for gap in GAPS:
        a, b = _gapped(rng, 1040, gap)
        pairs += [(a, b), (b, a)]
    pairs += _few_columns(rng, 1100) + [(b, a) for a, b in _few_columns(rng, 1030)]
    w = _workload(pairs, mode, go)
    cells, side = aln.aln_batch_route(w.n_pairs, aln.TRACEBACK)
    assert all(len(a) > side or len(b) > side or len(a) * len(b) >= cells for a, b in pairs)
    bad = compare(w, *run_gpu(w, aln.TRACEBACK, config=aln.BatchConfig(wf_group=group)), *run_oracle(w, True), "codes")
    assert not bad, bad[:3]
    gres, _ = run_gpu(w, aln.SCORE_ONLY, config=aln.BatchConfig(wf_min_cells=1, wf_group=group))
    ores, _ = run_oracle(w, False)
    bad = compare(w, gres, None, ores, None, "scores")
    assert not bad, bad[:3]
