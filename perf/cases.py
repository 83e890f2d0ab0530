"""The calls whose speed this repository watches: what its users have the aligner do, by size and kind.

Each case is one call of a public entry point on sequences that are already on the device:

  kind "pair"     LongAligner.run: one pair, scored or traced back;
  kind "batch"    BatchAligner.run: many pairs in one call, scored or traced back;
  kind "retrace"  aln_traceback: the CIGARs of pairs whose scores an earlier call found.

Schemes and length ranges are those of the benchmark's workloads (bench.py, synth/): 1000-letter global
pairs, long local DNA pairs, read/window pairs, and uneven protein batches, with the batch sizes that a
whole data set, a screening pass or one batch of the serving loop brings.
"""
import math

import numpy as np
import torch

import paper_2002_04561_amd as aln

DEVICE = "cuda"

# mode, alphabet, match, mismatch, gap open, gap extend (match None: a seeded substitution table)
SCHEMES = {
    "dna_global_linear": (aln.GLOBAL, 4, 2, -1, 0, -1),
    "dna_global_affine": (aln.GLOBAL, 4, 2, -3, -3, -1),
    "dna_local": (aln.LOCAL, 4, 2, -3, -3, -1),
    "reads": (aln.SEMIGLOBAL, 4, 1, -4, -5, -2),
    "protein": (aln.LOCAL, 20, None, None, -11, -1),
}
# Integer operations per cell of Eqs. (1)-(5): every two-input add or max and the substitution lookup once.
OPS = {"dna_global_linear": 5, "dna_global_affine": 10, "dna_local": 12, "reads": 10, "protein": 12}

READ_PAD = 64        # a read's window is this much longer than the read
# CIGAR words kept per pair of a batch: reads have few indels, fragments about one gap per hundred letters.
CIGAR_WORDS = {"reads": 64, "dna_global_affine": 1024, "dna_local": 1024}


def listed():
    return [
        # The paper's C example: one short pair, score and CIGAR.  The smallest call, all latency.
        dict(name="pair_1k_trace", kind="pair", scheme="dna_global_linear", n=1000, m=1000, trace=True),
        # A long genome pair, score and end cell only.
        dict(name="pair_262k_score", kind="pair", scheme="dna_local", n=262144, m=262144, trace=False),
        # A genome segment pair with its CIGAR (above 2^24 cells: traced back in linear space).
        dict(name="pair_64k_trace", kind="pair", scheme="dna_local", n=65536, m=65011, trace=True),
        # One batch of the serving loop's read class.
        dict(name="reads_400_trace", kind="batch", scheme="reads", pairs=400, lo=100, hi=250, trace=True),
        # A sequencing run's share of short reads against their windows, CIGAR for every read.
        dict(name="reads_1m_trace", kind="batch", scheme="reads", pairs=1 << 20, lo=100, hi=250, trace=True),
        # Screening: scores of candidate windows, no CIGARs.
        dict(name="reads_100k_score", kind="batch", scheme="reads", pairs=100003, lo=100, hi=250, trace=False),
        # CIGARs of the reads that a screening pass kept.
        dict(name="reads_20k_retrace", kind="retrace", scheme="reads", pairs=20011, lo=100, hi=250, trace=True),
        # Short peptides against each other: many small local pairs over 20 letters.
        dict(name="peptides_200k_score", kind="batch", scheme="protein", pairs=200003, lo=16, hi=128, trace=False),
        # One batch of the serving loop's protein class, with the routing that loop gives it.
        dict(name="protein_250_score", kind="batch", scheme="protein", pairs=250, lo=64, hi=16384, trace=False,
             min_cells=1),
        # A protein database chunk: very uneven lengths, scores and end cells.
        dict(name="protein_16k_score", kind="batch", scheme="protein", pairs=16384, lo=64, hi=16384, trace=False),
        # A handful of long pairs in one call (the serving loop's long class).
        dict(name="long_8_score", kind="batch", scheme="dna_local", pairs=8, lo=14000, hi=18000, trace=False),
        # Assembled fragments of mixed sizes against their references, end to end, with CIGARs.
        dict(name="fragments_1500_trace", kind="batch", scheme="dna_global_affine", pairs=1500, lo=100, hi=6000,
             trace=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same families; sizes spread over each family's range, odd ones among them."""
    family = rng.choice(["pair_trace_small", "pair_score", "pair_trace_long", "reads_trace", "reads_score",
                         "reads_retrace", "peptides", "protein", "long_batch", "fragments"])
    if family == "pair_trace_small":
        scheme = rng.choice(["dna_global_linear", "dna_global_affine", "dna_local", "reads"])
        return dict(kind="pair", scheme=scheme, n=_log_int(rng, 200, 4000), m=_log_int(rng, 200, 4000), trace=True)
    if family == "pair_score":
        scheme = rng.choice(["dna_global_affine", "dna_local", "reads"])
        return dict(kind="pair", scheme=scheme, n=_log_int(rng, 1000, 200000), m=_log_int(rng, 1000, 200000),
                    trace=False)
    if family == "pair_trace_long":
        n = _log_int(rng, 5000, 100000)
        return dict(kind="pair", scheme=rng.choice(["dna_global_affine", "dna_local"]), n=n,
                    m=int(n * rng.uniform(0.9, 1.1)), trace=True)
    if family in ("reads_trace", "reads_score", "reads_retrace"):
        top = {"reads_trace": 800000, "reads_score": 800000, "reads_retrace": 100000}[family]
        lo = rng.randint(50, 150)
        return dict(kind="retrace" if family == "reads_retrace" else "batch", scheme="reads",
                    pairs=_log_int(rng, 100, top), lo=lo, hi=rng.randint(lo, 300), trace=family != "reads_score")
    if family == "peptides":
        return dict(kind="batch", scheme="protein", pairs=_log_int(rng, 5000, 400000), lo=rng.randint(8, 32),
                    hi=rng.randint(60, 160), trace=False)
    if family == "protein":
        case = dict(kind="batch", scheme="protein", pairs=_log_int(rng, 50, 12000), lo=64,
                    hi=_log_int(rng, 1000, 16384), trace=False)
        if case["pairs"] < 1000:
            case["min_cells"] = 1
        return case
    if family == "long_batch":
        hi = _log_int(rng, 4000, 30000)
        return dict(kind="batch", scheme="dna_local", pairs=rng.randint(2, 24), lo=int(hi * 0.8), hi=hi, trace=False)
    return dict(kind="batch", scheme=rng.choice(["dna_global_affine", "dna_local"]),
                pairs=_log_int(rng, 50, 1500), lo=100, hi=_log_int(rng, 800, 6000), trace=True)


# ----------------------------------------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------------------------------------
class _Rand:
    """Seeded draws on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEVICE)
        self.g.manual_seed(seed)

    def unit(self, k):
        return torch.rand(k, generator=self.g, device=DEVICE, dtype=torch.float64)

    def ints(self, lo, hi, k):
        """k integers in [lo, hi]."""
        return torch.randint(lo, hi + 1, (k,), generator=self.g, device=DEVICE, dtype=torch.int64)

    def letters(self, alphabet, k):
        return torch.randint(0, alphabet, (k,), generator=self.g, device=DEVICE, dtype=torch.uint8)

    def geometric(self, mean, k):
        if mean <= 1.0:
            return torch.ones(k, device=DEVICE, dtype=torch.int64)
        u = self.unit(k).clamp_(min=1e-12)
        return (torch.log(u) / math.log(1.0 - 1.0 / mean)).long() + 1


def _offsets(lens):
    off = torch.zeros(lens.numel() + 1, device=DEVICE, dtype=torch.int64)
    torch.cumsum(lens, 0, out=off[1:])
    return off


def _mutate(r, src, src_off, p_sub, p_indel, mean):
    """Mutated copies of the concatenated sequences src: substitutions with p_sub, and with p_indel an
    insertion of random letters or a deletion, half each, of geometric length.  Returns (codes, offsets)."""
    total = src.numel()
    u = r.unit(total)
    coin = r.unit(total)
    indel = u < p_indel
    ins, dele = indel & (coin < 0.5), indel & (coin >= 0.5)
    sub = (u >= p_indel) & (u < p_indel + p_sub)
    shift = r.ints(1, 3, total).to(torch.uint8)
    out = torch.where(sub, (src + shift) % 4, src)
    length = r.geometric(mean, total)
    edge = torch.zeros(total + 1, device=DEVICE, dtype=torch.int64)
    at = torch.nonzero(dele).flatten()
    edge.index_add_(0, at, torch.ones_like(at))
    edge.index_add_(0, torch.clamp(at + length[at], max=total), -torch.ones_like(at))
    count = torch.where(torch.cumsum(edge, 0)[:total] > 0, 0, 1) + torch.where(ins, length, 0)
    ends = torch.cumsum(count, 0)
    codes = r.letters(4, int(ends[-1]))
    kept = torch.nonzero(torch.cumsum(edge, 0)[:total] == 0).flatten()
    codes[ends[kept] - 1] = out[kept]  # inserted letters come before the kept one
    return codes, torch.cat([ends.new_zeros(1), ends])[src_off]


def _fit(r, codes, m):
    """codes cut or padded with random letters to m letters."""
    if codes.numel() >= m:
        return codes[:m].contiguous()
    return torch.cat([codes, r.letters(4, m - codes.numel())])


def _scoring(case, seed):
    mode, alphabet, match, mismatch, go, ge = SCHEMES[case["scheme"]]
    if match is not None:
        return aln.Scoring(mode, alphabet, go, ge, match=match, mismatch=mismatch)
    rng = np.random.default_rng(seed)
    t = np.triu(rng.integers(-4, 4, (alphabet, alphabet)), 1)
    t = t + t.T
    np.fill_diagonal(t, rng.integers(4, 12, alphabet))
    return aln.Scoring(mode, alphabet, go, ge, subst=t.astype(np.int8))


def _sequences(case, seed):
    """(q, q_off, s, s_off): concatenated letter codes and their offsets."""
    r = _Rand(seed)
    if case["kind"] == "pair":
        n, m = case["n"], case["m"]
        q = r.letters(4, n)
        if case["scheme"] == "dna_global_linear":
            s = r.letters(4, m)  # unrelated, as in the benchmark's 1000-letter pair
        else:
            codes, _ = _mutate(r, q, torch.tensor([0, n], device=DEVICE), 0.05, 0.01, 3.0)
            s = _fit(r, codes, m)
        return q, _offsets(torch.tensor([n], device=DEVICE)), s, _offsets(torch.tensor([m], device=DEVICE))
    pairs, lo, hi = case["pairs"], case["lo"], case["hi"]
    if case["scheme"] == "reads":
        length = r.ints(lo, hi, pairs)
        s_off = _offsets(length + READ_PAD)
        s = r.letters(4, int(s_off[-1]))
        src_off = _offsets(length)
        pair_of = torch.repeat_interleave(torch.arange(pairs, device=DEVICE), length)
        start = s_off[:-1] + r.ints(0, READ_PAD, pairs) - src_off[:-1]
        src = s[torch.arange(pair_of.numel(), device=DEVICE) + start[pair_of]]
        q, q_off = _mutate(r, src, src_off, 0.02, 0.005, 1.0)
        return q, q_off, s, s_off
    if case["scheme"] == "protein":
        span = math.log(hi / lo)
        n = torch.round(lo * torch.exp(r.unit(pairs) * span)).long()
        m = torch.round(lo * torch.exp(r.unit(pairs) * span)).long()
        q_off, s_off = _offsets(n), _offsets(m)
        return r.letters(20, int(q_off[-1])), q_off, r.letters(20, int(s_off[-1])), s_off
    span = math.log(hi / lo)
    q_off = _offsets(torch.round(lo * torch.exp(r.unit(pairs) * span)).long())
    q = r.letters(4, int(q_off[-1]))
    s, s_off = _mutate(r, q, q_off, 0.05, 0.01, 3.0)
    return q, q_off, s, s_off


def _longest(off):
    return max(int((off[1:] - off[:-1]).max()), 1)


def prepare(case, seed):
    q, q_off, s, s_off = _sequences(case, seed)
    scoring = _scoring(case, seed)
    flags = aln.TRACEBACK if case["trace"] else aln.SCORE_ONLY
    if case["kind"] == "pair":
        a = aln.LongAligner(scoring, q, s, flags)
        if a.cigar is not None:
            a.cigar.zero_()
        return dict(aligner=a)
    max_n, max_m = _longest(q_off), _longest(s_off)
    pairs = case["pairs"]
    words = CIGAR_WORDS.get(case["scheme"], 0)
    capacity = np.full(pairs, words, np.int64) if case["trace"] else None
    if case["kind"] == "batch":
        config = aln.BatchConfig(wf_min_cells=case["min_cells"]) if "min_cells" in case else None
        a = aln.BatchAligner(scoring, q, q_off, s, s_off, max_n, max_m, flags, cigar_capacity=capacity, config=config)
        if a.cigar is not None:
            a.cigar.zero_()
        return dict(aligner=a)
    # the forward scores that the screening call left behind
    fwd = aln.BatchAligner(scoring, q, q_off, s, s_off, max_n, max_m, aln.SCORE_ONLY)
    fwd.run()
    cigar_off = torch.arange(pairs + 1, device=DEVICE, dtype=torch.int64) * words
    nbytes = aln.aln_traceback_workspace_size(scoring, pairs, max_n, max_m)
    return dict(scoring=scoring, pairs=pairs, q=q, q_off=q_off, s=s, s_off=s_off, max_n=max_n, max_m=max_m,
                fwd=fwd.out, out=torch.empty_like(fwd.out), nbytes=nbytes, cigar_off=cigar_off,
                cigar=torch.zeros(pairs * words, device=DEVICE, dtype=torch.int32),
                workspace=torch.empty(max(nbytes, 256), device=DEVICE, dtype=torch.uint8))


def run(state):
    if "aligner" in state:
        a = state["aligner"]
        a.run()
        return (a.out,) if a.cigar is None else (a.out, a.cigar)
    st = aln.aln_traceback(state["scoring"], state["pairs"], state["q"], state["q_off"], state["s"], state["s_off"],
                           state["max_n"], state["max_m"], state["fwd"], state["out"], state["cigar"],
                           state["cigar_off"], state["workspace"], state["nbytes"])
    if st != 0:
        raise aln.AlnError(st, "aln_traceback")
    return state["out"], state["cigar"]


def work(case):
    """Sequences and offsets read once, a 32-byte result per pair and its CIGAR written once (one word per
    100 letters for reads, one per two letters between unrelated sequences, one per 25 between related
    ones); the operations of the recurrence for every cell, once."""
    if case["kind"] == "pair":
        pairs, letters, cells = 1, case["n"] + case["m"], float(case["n"]) * case["m"]
    else:
        pairs, lo, hi = case["pairs"], case["lo"], case["hi"]
        if case["scheme"] == "reads":
            mean = (lo + hi) / 2.0
            square = mean * mean + (hi - lo) ** 2 / 12.0
            letters, cells = pairs * (2 * mean + READ_PAD), pairs * (square + READ_PAD * mean)
        else:
            span = math.log(hi / lo) if hi > lo else 1.0
            mean = (hi - lo) / span if hi > lo else float(lo)
            square = (hi * hi - lo * lo) / (2 * span) if hi > lo else float(lo * lo)
            letters = 2 * mean * pairs
            cells = pairs * (mean * mean if case["scheme"] == "protein" else square)
    per_word = {"reads": 100, "dna_global_linear": 4}.get(case["scheme"], 50)
    nbytes = letters + 48 * pairs + (4 * letters / per_word if case["trace"] else 0)
    return {"bytes": int(nbytes), "flops": int(cells * OPS[case["scheme"]])}


# ----------------------------------------------------------------------------------------------------------
# The same alignments in plain numpy, 64-bit, from the definition.
# ----------------------------------------------------------------------------------------------------------
_NEG = -(1 << 40)


def _align(mode, sigma, go, ge, q, s, trace):
    """One pair: (score, q_begin, q_end, s_begin, s_end, CIGAR words)."""
    n, m = len(q), len(s)
    col = np.arange(m + 1, dtype=np.int64)
    H, E, F = (np.full((n + 1, m + 1), _NEG, dtype=np.int64) for _ in range(3))
    H[0] = 0
    H[:, 0] = 0
    if mode == aln.GLOBAL:
        H[0, 1:] = go + col[1:] * ge
        H[1:, 0] = go + np.arange(1, n + 1) * ge
    for i in range(1, n + 1):
        E[i, 1:] = np.maximum(E[i - 1, 1:] + ge, H[i - 1, 1:] + go + ge)
        h = np.maximum(H[i - 1, :-1] + sigma[q[i - 1]][s], E[i, 1:])
        if mode == aln.LOCAL:
            h = np.maximum(h, 0)
        # a gap that opens where another horizontal gap ends is never better than extending it, so F needs
        # only the cells' values without F: a running maximum along the row
        base = np.concatenate([H[i, :1], h]) - col * ge
        F[i, 1:] = np.maximum.accumulate(base)[:-1] + go + col[1:] * ge
        H[i, 1:] = np.maximum(h, F[i, 1:])
    if mode == aln.GLOBAL:
        i, j = n, m
    elif mode == aln.LOCAL:
        i, j = divmod(int(np.argmax(H)), m + 1)  # the first maximum in row-major order
    else:
        j = m
        i = int(np.argmax(H[:, m]))
        k = int(np.argmax(H[n]))
        if H[n, k] > H[i, m] or (H[n, k] == H[i, m] and i == n):
            i, j = n, k
    score = int(H[i, j])
    if mode == aln.LOCAL and score == 0:
        i = j = 0
    ends = (i, j)
    if not trace:
        return score, -1, ends[0], -1, ends[1], []
    runs, gap = [], 0

    def step(op, k=1):
        if runs and runs[-1][1] == op:
            runs[-1][0] += k
        else:
            runs.append([k, op])

    while True:
        if gap == 0:
            if i == 0 or j == 0:
                if mode == aln.GLOBAL and i + j > 0:
                    step(aln.CIGAR_D if j else aln.CIGAR_I, i + j)
                    i = j = 0
                break
            h = H[i, j]
            if mode == aln.LOCAL and h == 0:
                break
            if h == H[i - 1, j - 1] + sigma[q[i - 1], s[j - 1]]:
                step(aln.CIGAR_M)
                i, j = i - 1, j - 1
                continue
            gap = 1 if h == E[i, j] else 2
        if gap == 1:
            step(aln.CIGAR_I)
            if E[i, j] == H[i - 1, j] + go + ge or i == 1:
                gap = 0
            i -= 1
        else:
            step(aln.CIGAR_D)
            if F[i, j] == H[i, j - 1] + go + ge or j == 1:
                gap = 0
            j -= 1
    return score, i, ends[0], j, ends[1], [(k << 4) | op for k, op in reversed(runs)]


def exact(case, seed):
    """What run returns, or None where numpy would take too long."""
    if case["kind"] == "pair":
        rows, cells = case["n"], case["n"] * case["m"]
    else:
        rows, cells = case["pairs"] * case["hi"], case["pairs"] * case["hi"] * (case["hi"] + READ_PAD)
    if rows > 150000 or cells > 2e7:
        return None
    q, q_off, s, s_off = (x.cpu().numpy() for x in _sequences(case, seed))
    sc = _scoring(case, seed)
    if sc.subst is not None:
        sigma = sc.subst.astype(np.int64)
    else:
        sigma = np.full((4, 4), sc.mismatch, dtype=np.int64)
        np.fill_diagonal(sigma, sc.match)
    pairs = len(q_off) - 1
    results = np.zeros((pairs, 8), dtype=np.int64)
    words = []
    for k in range(pairs):
        a, b = q[q_off[k]:q_off[k + 1]], s[s_off[k]:s_off[k + 1]]
        score, qb, qe, sb, se, cig = _align(sc.mode, sigma, sc.gap_open, sc.gap_extend, a, b, case["trace"])
        results[k, :6] = score, qb, qe, sb, se, len(cig)
        room = len(a) + len(b) + 1 if case["kind"] == "pair" else CIGAR_WORDS.get(case["scheme"], 0)
        if len(cig) > room:
            return None  # truncated: run says so, and keeps no CIGAR
        words.append(np.array(cig + [0] * (room - len(cig)), dtype=np.int64))
    out = torch.from_numpy(results.reshape(-1))
    return (out, torch.from_numpy(np.concatenate(words))) if case["trace"] else (out,)
