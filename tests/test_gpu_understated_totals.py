"""Traceback batches whose total_q / total_s lie below the real sums: the code arena, sized from them, has no room for the
large pairs, which the planner then leaves to the small-pair kernels.  Their workspace holds pairs up to 1024 letters a
side: a longer one is flagged ALN_RES_TOO_LONG, by the kernel of one wave per pair (short batch) as by those of one pair per
lane (long batch), and every other pair comes back exact."""
import numpy as np
import pytest

import synth
from helpers import run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("copies,kernel", [(2, "batch_wave_traceback"), (44000, "batch_i16_traceback")])
def test_understated_totals_traceback(gpu, mode, copies, kernel):
    import torch

    import paper_2002_04561_amd as aln
    rng = np.random.default_rng(43)
    lens = [(1500, 1400), (1025, 300), (300, 1025), (1024, 1024), (600, 500)]
    lens += [(12, 9), (7, 0), (20, 11), (1, 3), (15, 15), (9, 18)] * copies
    qs = [rng.integers(0, 4, n, dtype=np.uint8) for n, _ in lens]
    ss = [rng.integers(0, 4, m, dtype=np.uint8) for _, m in lens]
    w = synth.Workload("understated", mode, 4, -3, -1, *synth.pack(qs), *synth.pack(ss), match=2, mismatch=-3, traceback=True)
    q, qo, s, so = aln.to_device(w)
    ba = aln.BatchAligner(aln.scoring_of(w), q, qo, s, so, 1500, 1400, aln.TRACEBACK, total_q=64, total_s=64)
    aln.aln_profile_enable(True)
    aln.aln_profile_reset()
    ba.run()
    torch.cuda.synchronize()
    ran = aln.aln_profile_read()
    aln.aln_profile_enable(False)
    assert kernel in ran, ran
    res, cig = ba.results(), ba.cigars()
    long = np.array([n > 1024 or m > 1024 for n, m in lens])
    assert (res["flags"][long] == aln.RES_TOO_LONG).all(), res["flags"][:5]
    assert not res["flags"][~long].any()
    assert not res["score"][long].any() and not res["cigar_len"][long].any()
    ores, ocig = run_oracle(w, True)
    for f in ("score", "q_begin", "q_end", "s_begin", "s_end"):
        assert (res[f] == ores[f])[~long].all(), f
    assert [c for c, x in zip(cig, long) if not x] == [c for c, x in zip(ocig, long) if not x]
