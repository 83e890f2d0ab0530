"""Which kernel runs a traceback batch's small pairs goes by the pairs' own lengths where the call's bounds lie far above them:
20,000 pairs of 8..30 letters run one per lane under every bound (a loose one once sent them one per wave, up to 8 times slower),
and one per wave once they hold a pair that would keep a lane busy for longer; the same for aln_traceback.  Both kernels are
launched and one has no pairs, so the route shows in their times.  Results equal the oracle's either way, in replays of a
graph too."""
import numpy as np
import pytest

import synth
from helpers import compare, run_oracle

pytestmark = pytest.mark.gpu
N = 20000


def _workload(mode, outlier):
    rng = np.random.default_rng(50 + mode)
    lens = rng.integers(8, 31, (N, 2))
    if outlier:
        lens[N // 3] = (480, 500)
    qo = np.concatenate([[0], np.cumsum(lens[:, 0])]).astype(np.int64)
    so = np.concatenate([[0], np.cumsum(lens[:, 1])]).astype(np.int64)
    q, s = rng.integers(0, 4, int(qo[-1]), dtype=np.uint8), rng.integers(0, 4, int(so[-1]), dtype=np.uint8)
    return synth.Workload("route", mode, 4, -3, -1, q, qo, s, so, match=2, mismatch=-3, traceback=True)


def _times(call):
    """{kernel: ms} of the fastest of three calls."""
    import torch

    import paper_2002_04561_amd as aln
    best = {}
    call()
    for _ in range(3):
        aln.aln_profile_enable(True)
        aln.aln_profile_reset()
        call()
        torch.cuda.synchronize()
        for k, (_, ms) in aln.aln_profile_read().items():
            best[k] = min(ms, best.get(k, ms))
        aln.aln_profile_enable(False)
    return best


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("outlier", [False, True], ids=["small", "outlier"])
@pytest.mark.parametrize("bits", [16, 32])
def test_batches(gpu, mode, outlier, bits):
    import torch

    import paper_2002_04561_amd as aln
    w = _workload(mode, outlier)
    q, qo, s, so = aln.to_device(w)
    ba = aln.BatchAligner(aln.scoring_of(w), q, qo, s, so, 512, 512, aln.TRACEBACK | (aln.FORCE_INT32 if bits == 32 else 0))
    t = _times(ba.run)
    lanes, waves = t["batch_i%d_traceback" % bits], t["batch_wave_traceback"]
    assert (waves > lanes) == outlier, t
    ores, ocig = run_oracle(w, True)
    bad = compare(w, ba.results(), ba.cigars(), ores, ocig, "route")
    assert not bad, bad[:3]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ba.run()
    for _ in range(3):
        ba.out.zero_()
        ba.cigar.zero_()
        g.replay()
        torch.cuda.synchronize()
        bad = compare(w, ba.results(), ba.cigars(), ores, ocig, "replay")
        assert not bad, bad[:3]


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["global", "local", "semi"])
@pytest.mark.parametrize("outlier", [False, True], ids=["small", "outlier"])
def test_traceback_from_ends(gpu, mode, outlier):
    import torch

    import paper_2002_04561_amd as aln
    w = _workload(mode, outlier)
    if outlier:
        # its two sequences alike, so that its alignment ends far out in every mode
        k = N // 3
        w.s[w.s_off[k]:w.s_off[k] + 480] = w.q[w.q_off[k]:w.q_off[k] + 480]
    q, qo, s, so = aln.to_device(w)
    sc = aln.scoring_of(w)
    fwd = aln.BatchAligner(sc, q, qo, s, so, 512, 512, aln.SCORE_ONLY)
    fwd.run()
    cap = np.concatenate([[0], np.cumsum(np.diff(w.q_off) + np.diff(w.s_off))]).astype(np.int64)
    coff = torch.from_numpy(cap).cuda()
    cig = torch.zeros(int(cap[-1]), dtype=torch.int32, device="cuda")
    out = torch.empty_like(fwd.out)
    nbytes = aln.aln_traceback_workspace_size(sc, N, 512, 512)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")

    def call():
        assert aln.aln_traceback(sc, N, q, qo, s, so, 512, 512, fwd.out, out, cig, coff, ws, nbytes) == 0

    t = _times(call)
    assert (t["batch_wave_traceback_from_end"] > t["batch_i32_traceback_from_end"]) == outlier, t
    res = out.cpu().numpy().view(aln.RESULT_DTYPE)
    words = cig.cpu().numpy().view(np.uint32)
    gcig = [[(int(x) >> 4, int(x) & 15) for x in words[cap[k]:cap[k] + res["cigar_len"][k]]] for k in range(N)]
    bad = compare(w, res, gcig, *run_oracle(w, True), "ends")
    assert not bad, bad[:3]
