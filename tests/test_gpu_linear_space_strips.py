"""Linear-space tracebacks of subjects about one tile (2048 columns) long: up to one tile across a segment is relaxed in one
phase, past it in bands around the walk.  Queries of one and of several segments (a segment is one tile row of 1024 rows here),
with a long gap in either sequence.  Equal to the oracle's canonical traceback."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [synth.GLOBAL, synth.LOCAL, synth.SEMIGLOBAL], ids=["global", "local", "semiglobal"])
@pytest.mark.parametrize("n", [1, 900, 3300])
@pytest.mark.parametrize("m", [1, 2047, 2048, 2049])
def test_subjects_of_one_tile(gpu, mode, n, m):
    import torch

    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(n + m)
    q = rng.integers(0, 4, n, dtype=np.uint8)
    s = rng.integers(0, 4, m, dtype=np.uint8)
    k = min(n, m) * 2 // 5
    s[:k] = q[:k]  # the common ends lie far from one diagonal
    s[m - k:] = q[n - k:]
    aln.aln_set_traceback_budget(64 << 10)
    try:
        la = aln.LongAligner(aln.Scoring(mode, 4, -4, -1, match=3, mismatch=-3), torch.from_numpy(q).cuda(),
                             torch.from_numpy(s).cuda(), aln.TRACEBACK | aln.LINEAR_SPACE)
        la.run()
        torch.cuda.synchronize()
    finally:
        aln.aln_set_traceback_budget(0)
    g = la.result()
    r = oracle.align(oracle.Scoring.simple(mode, 4, 3, -3, -4, -1), q, s, traceback=True, impl="checkpointed")
    got = tuple(int(g[f]) for f in ("score", "q_begin", "q_end", "s_begin", "s_end", "flags")) + (la.cigar_runs(),)
    assert got == (r.score, r.q_begin, r.q_end, r.s_begin, r.s_end, 0, r.cigar)
