"""Tracebacks whose walks leave the diagonal: a related pair with one inserted block around the sizes of the walk's windows (its
window along the diagonal reaches 11 cells right and 14 left, its rectangles are 32 and 128 wide and 128 and 32 rows high), pairs
of very different lengths, and subjects of a few letters, where a band's first columns and its last fall into one step; on the
kernel of one wave per pair and on the band wavefront, equal to the oracle's."""
import numpy as np
import pytest

import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _pairs(mode):
    rng = np.random.default_rng(mode)
    qs, ss = [], []
    for gap in (10, 11, 12, 13, 14, 15, 16, 31, 32, 33, 64, 65, 127, 128, 129, 300):
        a, ins = rng.integers(0, 4, 260, dtype=np.uint8), rng.integers(0, 4, gap, dtype=np.uint8)
        b = np.concatenate([a[:131], ins, a[131:]])
        qs += [a, b]
        ss += [b, a]
    for n, m in ((700, 60), (60, 700), (600, 1), (1, 600), (520, 2), (300, 66), (513, 63), (400, 64), (64, 65)):
        qs.append(rng.integers(0, 4, n, dtype=np.uint8))
        ss.append(rng.integers(0, 4, m, dtype=np.uint8))
    return qs, ss


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("go", [0, -3], ids=["linear", "affine"])
@pytest.mark.parametrize("wavefront", [False, True], ids=["wave_per_pair", "wavefront"])
def test_walks_off_the_diagonal(gpu, mode, go, wavefront):
    import paper_2002_04561_amd as aln
    qs, ss = _pairs(mode)
    q, qo = synth.pack(qs)
    s, so = synth.pack(ss)
    w = synth.Workload("gaps", mode, 4, go, -1, q, qo, s, so, match=5, mismatch=-4, traceback=True)
    bad = compare(w, *run_gpu(w, aln.TRACEBACK, config=aln.BatchConfig(wf_min_cells=1) if wavefront else None),
                  *run_oracle(w, True), "gaps")
    assert not bad, bad[:3]
