"""Linear-space tracebacks whose walk leaves every band of tiles that a segment relaxes again: bands reach 1024, 4096 and 16384
columns to either side of the walk's diagonal, each around the cell where the walk left the one before, and after the third
every tile left of the walk is relaxed.  A subject with 30,000 letters inserted in the middle of a 3000-letter query,
global, takes one horizontal gap of that length (with affine gaps), from column 31,500 to column 1500: past the three bands
together, whose left edges lie at columns 28,672, 22,528 and 4096.  With 3,000 and 12,000 letters the second and the
third band hold it.  Equal to the oracle's canonical traceback (its own, from stored rows)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gap", [(0, -1), (-3, -1)], ids=["linear", "affine"])
@pytest.mark.parametrize("inserted", [3000, 12000, 30000])
@pytest.mark.parametrize("alphabet", [4, 20], ids=["register_profile", "table_profile"])
def test_gap_past_the_bands(gpu, gap, inserted, alphabet):
    import torch

    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(inserted + alphabet)
    go, ge = gap
    q = rng.integers(0, alphabet, 3000, dtype=np.uint8)
    s = np.concatenate([q[:1500], rng.integers(0, alphabet, inserted, dtype=np.uint8), q[1500:]])
    aln.aln_set_traceback_budget(64 << 10)  # segments of one tile row: 1024 rows
    try:
        la = aln.LongAligner(aln.Scoring(synth.GLOBAL, alphabet, go, ge, match=3, mismatch=-3), torch.from_numpy(q).cuda(),
                             torch.from_numpy(s).cuda(), aln.TRACEBACK | aln.LINEAR_SPACE)
        la.run()
        torch.cuda.synchronize()
    finally:
        aln.aln_set_traceback_budget(0)
    g = la.result()
    r = oracle.align(oracle.Scoring.simple(synth.GLOBAL, alphabet, 3, -3, go, ge), q, s, traceback=True, impl="checkpointed")
    got = tuple(int(g[f]) for f in ("score", "q_begin", "q_end", "s_begin", "s_end", "flags")) + (la.cigar_runs(),)
    assert got == (r.score, r.q_begin, r.q_end, r.s_begin, r.s_end, 0, r.cigar)
    if go < 0:
        assert max(length for length, op in r.cigar if op == oracle.OP_D) >= inserted - 100
