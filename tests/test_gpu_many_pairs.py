"""Batches of many small pairs on the band wavefront: one band a pair, which the waves take in turn, and pair counts
around the planner's chunks, with empty pairs and two-band pairs mixed in: all equal to the oracle's."""
import numpy as np
import pytest

import synth
from helpers import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("n_pairs", [1, 255, 256, 257, 5000, 70001])
@pytest.mark.parametrize("two_bands", [False, True], ids=["one_band", "mixed"])
def test_many_pairs(gpu, mode, n_pairs, two_bands):
    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(n_pairs + mode)
    top = 20 if n_pairs > 1000 else 256
    lens = rng.integers(0, top + 1, (n_pairs, 2))
    lens[-1] = (top, top)
    if two_bands:
        lens[rng.integers(0, n_pairs, 3)] = (257, 30)
    q_off = np.concatenate([[0], np.cumsum(lens[:, 0])]).astype(np.int64)
    s_off = np.concatenate([[0], np.cumsum(lens[:, 1])]).astype(np.int64)
    q = rng.integers(0, 4, int(q_off[-1]), dtype=np.uint8)
    s = rng.integers(0, 4, int(s_off[-1]), dtype=np.uint8)
    w = synth.Workload("many", mode, 4, -3, -1, q, q_off, s, s_off, match=2, mismatch=-3)
    gres, _ = run_gpu(w, aln.SCORE_ONLY, config=aln.BatchConfig(wf_min_cells=1, wf_group=1))
    ores, _ = run_oracle(w, False)
    bad = compare(w, gres, None, ores, None, "many")
    assert not bad, bad[:3]
