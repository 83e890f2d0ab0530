"""Semi-global optima in row n: the query occurs in the subject again and again, so the row's best score comes back at many columns
and the first of them wins.  Every place of row n in a lane and in a band, copies that start at every column of a group of 4,
first and last columns, transposed pairs and both engines, with and without CIGARs: equal to the oracle's."""
import numpy as np
import pytest

import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

ROWS = (1, 2, 3, 4, 5, 7, 63, 64, 65, 253, 254, 255, 256, 257, 258, 259, 511, 513)


def _workload(seed, go):
    rng = np.random.default_rng(seed)
    qs, ss = [], []
    for n in ROWS:
        a = rng.integers(0, 4, n, dtype=np.uint8)
        for gap in range(4):
            parts = []
            for _ in range(3):
                parts += [rng.integers(0, 4, int(rng.integers(0, 9)) + gap, dtype=np.uint8), a]
            qs += [a, a, a]
            # the last copy ends at column m, stops one short of it, or is followed by other letters
            s = np.concatenate(parts)
            ss += [s, s[:-1], np.concatenate([s, rng.integers(0, 4, 70 + gap, dtype=np.uint8)])]
    q, qo = synth.pack(qs)
    s, so = synth.pack(ss)
    return synth.Workload("last_row", synth.SEMIGLOBAL, 4, go, -1, q, qo, s, so, match=2, mismatch=-3, traceback=True)


@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
@pytest.mark.parametrize("group", [1, 4], ids=["bands_alone", "bands_in_groups"])
@pytest.mark.parametrize("orient", [-1, 1], ids=["as_given", "longer_along_rows"])
def test_scores(gpu, go, group, orient):
    import paper_2002_04561_amd as aln
    w = _workload(60, go)
    gres, _ = run_gpu(w, aln.SCORE_ONLY, config=aln.BatchConfig(wf_min_cells=1, wf_group=group, wf_orient=orient))
    ores, _ = run_oracle(w, False)
    bad = compare(w, gres, None, ores, None, "scores")
    assert not bad, bad[:3]


@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
def test_cigars(gpu, go):
    import paper_2002_04561_amd as aln
    w = _workload(61, go)
    bad = compare(w, *run_gpu(w, aln.TRACEBACK), *run_oracle(w, True), "cigars")
    assert not bad, bad[:3]
