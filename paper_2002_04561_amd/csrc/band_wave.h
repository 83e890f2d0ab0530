// What one wave does with a band of 64 x R rows beyond the recurrence of band.h: its letters, its start, the optimum it
// tracks and its result.  Shared by the band wavefront (wf_i32.hip) and the one-wave-per-pair kernel (batch_wave.hip).
#pragma once
#include "band.h"

extern "C" __device__ __attribute__((const)) int __ockl_wfred_max_i32(int);  // maximum over the wave

namespace mialign {

// Local alignment: every lane keeps the best score its rows have seen (bs) and the first cell, by row and then by
// column, that reached it.  The pair's optimum -- the first cell in (score, i, j) order -- scores at least as high
// as every real cell, so once per block each lane's running value is raised to the largest score seen so far minus
// one (ties still pass, also for transposed pairs, whose caller rows run along the band): the best of the
// band's top-row inputs, which are cells of an earlier row, and the best its own lanes have recorded.  Lanes then
// record only cells that may still be the optimum.  On related sequences the top row stays ahead of the values
// that climb towards the diagonal inside the band; on unrelated ones the band's best over all its rows is
// rarely beaten.  A raised value never wins: it is below a real cell, which some band records or beats.  top_h
// is the score of the lane's top-row input, or 0 (at most H = 0) on lanes without one.  Rows past n and columns
// outside 1..m need no mask: with gap scores <= 0 and a negative pad letter their values come from real cells'
// minus penalties, or from the floor H = 0, so they never reach the optimum.  Every lane of the wave calls
// this; it returns the raised floor, which no lane's bs is below.
__device__ __forceinline__ int raise_local_floor(int32_t& bs, int32_t top_h) {
  const int32_t fl = __ockl_wfred_max_i32(max(bs, top_h)) - 1;
  bs = max(bs, fl);
  return fl;
}

// Per lane, a where the lane's bit of mask is set, else b: one v_cndmask.  The select is the compiler's own, which keeps the wait
// states that an SGPR written by a VALU instruction (a comparison, v_readlane) needs before a VALU instruction reads it;
// inline asm does not get them.  The mask stays a mask: the compiler cannot tell which comparison it came from and branch on it.
__device__ __forceinline__ int mask_select(unsigned long long mask, int a, int b) {
  return __builtin_amdgcn_inverse_ballot_w64(mask) ? a : b;
}

// (score, i, j) order of optima: larger score, then smaller i, then smaller j.
__device__ __forceinline__ bool better(int s1, int i1, int j1, int s2, int i2, int j2) {
  return s1 > s2 || (s1 == s2 && (i1 < i2 || (i1 == i2 && j1 < j2)));
}

// Per wave, the letters of the columns in flight as profile indices: 64 columns before the block, then the block's
// own (and the 8 columns that the last groups look ahead to, never used).  Step t of the block at tb has lane l
// at column t - l + 1, so a lane reads 4 consecutive entries a group.
template <int BLK>
struct LetterWindow {
  int v[64 + BLK + 12];
  // old: the letter of column tb - 63 + lane; cur: lane < BLK, of column tb + 1 + lane
  __device__ __forceinline__ void put(int lane, int old, int cur) {
    v[lane] = old;
    if (BLK >= 64 || lane < BLK) v[64 + lane] = cur;
  }
  __device__ __forceinline__ void get(int lane, int g4, int (&c)[4]) const {
    const int* p = v + 64 - lane + 4 * g4;
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = p[u];
  }
  __device__ __forceinline__ void clear_tail(int lane) {
    if (lane < 12) v[64 + BLK + lane] = 0;
  }
};

// What a lane keeps of its best cells.  Local: the best score, the group of 4 steps that first reached it (its first
// column and its cells' values), and the largest score known anywhere in the band minus one.  Otherwise: the best score in
// column m and its row (kj), and the best of row n.
template <int R>
struct BandBest {
  int32_t bs = kNeg32;
  int floor = -1;
  int kj = INT32_MIN;
  int32_t kv[4][R];
  int thr = INT32_MAX;  // row n, in its lane: the best H(n, j) + go - rn * ge, H(n, 0) = 0 first
  int browj = INT32_MIN;  // the first column of the group that reached it, and the row's values there
  int rv[4] = {};
};

// The first cell that holds a group's largest value v(u, r) + (r + u) * ge: by row and then by column, or (BY_COL) by
// column and then by row.
template <int R, bool BY_COL>
__device__ __forceinline__ void first_best(const KParams& P, const int32_t (&v)[4][R], int& br, int& bu) {
  int32_t best = INT32_MIN;
  br = bu = 0;
#pragma unroll
  for (int a = 0; a < (BY_COL ? 4 : R); ++a)
#pragma unroll
    for (int b = 0; b < (BY_COL ? R : 4); ++b) {
      const int r = BY_COL ? b : a, u = BY_COL ? a : b;
      const int32_t x = v[u][r] + (r + u) * P.ge;
      if (x > best) {
        best = x;
        br = r;
        bu = u;
      }
    }
}

// After 4 steps of a local band (columns j0 .. j0 + 3, floor0: the floor of the lane's first row at column j0).
// A group matters only where some cell beats the floor, and no cell does unless the sums below do: g of every
// cell flows down into E~ of the lane's last row or is that row's g, and that row's F~ holds the g of its earlier
// columns, so their maximum is at least every g of the group; a cell that beats the floor has
// g > floor0 + floor + go.  With a linear gap the last cell is itself at least every cell.  That costs 4 issue
// slots for 16 cells; comparing each row's maximum took 12.
// Where the test passes, the exact best of the group is the largest of the anti-diagonals' maxima (whose cells share
// a bias).  A lane that improves keeps the group's values, 16 selects; its cell is looked up at the band's end.
// One long pair's bands improve in a hundred groups or more where they meet the alignment's diagonal, and every step a
// band spends there delays each band below it: looking the cell up at once took 45.5 ms on 262144^2 related DNA.
template <bool AFFINE, int R>
__device__ __forceinline__ void track_local(const KParams& P, const BandLane<R>& L, const BandGroup<R>& G, int floor0,
                                            int j0, bool flip, BandBest<R>& B) {
  static_assert(R == 4, "the anti-diagonals of a 4 x 4 group");
  int x;
  if (AFFINE)
    x = max(max3i(max3i(G.oe[0], G.oe[1], G.oe[2]), G.oe[3], L.f[R - 1]), L.g[R - 1]);
  else
    x = G.v[3][R - 1];
  if (__builtin_amdgcn_ballot_w64(x - floor0 > B.floor + P.go) == 0) return;
  const auto& v = G.v;
  const int t1 = max(v[0][1], v[1][0]), t2 = max3i(v[0][2], v[1][1], v[2][0]);
  const int t3 = max(max3i(v[0][3], v[1][2], v[2][1]), v[3][0]);
  const int t4 = max3i(v[1][3], v[2][2], v[3][1]), t5 = max(v[2][3], v[3][2]);
  int32_t mk = max3i(v[0][0], t1 + P.ge, t2 + 2 * P.ge);
  mk = max3i(mk, t3 + 3 * P.ge, t4 + 4 * P.ge);
  mk = max3i(mk, t5 + 5 * P.ge, v[3][3] + 6 * P.ge);
  mk -= floor0 + P.go;
  const unsigned long long over = __builtin_amdgcn_ballot_w64(mk > B.floor);
  if (over == 0) return;
  unsigned long long up = over & __builtin_amdgcn_ballot_w64(mk > B.bs);
  // an equal cell replaces the lane's where its row is smaller (of a flipped pair, whose rows are the call's columns,
  // never: its column is larger)
  unsigned long long tie = over & __builtin_amdgcn_ballot_w64(mk == B.bs);
  if (tie && !flip) {
    int r1, u1, r0, u0;
    first_best<R, false>(P, v, r1, u1);
    first_best<R, false>(P, B.kv, r0, u0);
    up |= tie & __builtin_amdgcn_ballot_w64(r1 < r0);
  }
  if (up == 0) return;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int u = 0; u < 4; ++u) B.kv[u][r] = mask_select(up, v[u][r], B.kv[u][r]);
  B.kj = mask_select(up, j0, B.kj);
  B.bs = mask_select(up, mk, B.bs);
  // one lane's new best raises the floor of the whole band at once
  B.floor = max(B.floor, __builtin_amdgcn_readlane(mk, (int)__builtin_ctzll(up)) - 1);
}

// The kept group's first best cell: its row among the lane's and its column (-1: none kept).
template <int R>
__device__ __forceinline__ void resolve_kept(const KParams& P, const BandBest<R>& B, bool flip, int& br, int& bj) {
  br = bj = -1;
  if (B.kj == INT32_MIN) return;
  int u;
  if (flip)
    first_best<R, true>(P, B.kv, br, u);
  else
    first_best<R, false>(P, B.kv, br, u);
  bj = B.kj + u;
}

// The semi-global band that holds row n, which is one lane's row rn (elsewhere rn is outside 0 .. R - 1): its cells in columns
// 1..m.  Only that lane's threshold is ever passed.
template <int R>
__device__ __forceinline__ void last_row_start(const KParams& P, int rn, BandBest<R>& B) {
  B.thr = rn >= 0 && rn < R ? P.go - rn * P.ge : INT32_MAX;
}

// After 4 steps of that band (row_n: row n's index in the band).  As above, the row's F~ and last g (linear: its last cell) bound
// the group's cells, so most groups cost a maximum and a select per row and a compare.  A group that passes has its exact best
// compared, and one that improves leaves the row's four values, whose first best column is looked up at the band's end.  Which of
// a lane's rows it is, is the same for the whole wave: the picks' masks are scalars that stay.
// This band comes last, so its steps are at the end of every chain, and between related sequences with linear gaps nearly every
// group improves: comparing the four cells in turn took 4.50 ms for 30000 x 30000 such letters where this takes 4.00 (affine gaps
// 4.38 and 4.15; 200 x 20000, where few groups improve, 1.92 and 1.74).
template <bool AFFINE, int R>
__device__ __forceinline__ void track_last_row(const KParams& P, const BandLane<R>& L, const BandGroup<R>& G, int floor0,
                                               int m, int row_n, int j0, BandBest<R>& B) {
  static_assert(R == 4, "a row is picked by two bits of its index");
  const unsigned long long b0 = row_n & 1 ? ~0ull : 0ull, b1 = row_n & 2 ? ~0ull : 0ull;
  auto pick = [&](int x0, int x1, int x2, int x3) {
    return mask_select(b1, mask_select(b0, x3, x2), mask_select(b0, x1, x0));
  };
  int last[R];
#pragma unroll
  for (int r = 0; r < R; ++r) last[r] = AFFINE ? max(L.f[r], L.g[r]) : L.h[r];
  if (__builtin_amdgcn_ballot_w64(pick(last[0], last[1], last[2], last[3]) - floor0 > B.thr) == 0) return;
  int x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    x[u] = pick(G.v[u][0], G.v[u][1], G.v[u][2], G.v[u][3]) + u * P.ge;
    if (j0 + u < 1 || j0 + u > m) x[u] = INT32_MIN;
  }
  const int best = max(max3i(x[0], x[1], x[2]), x[3]);
  // (where a column is missing the others still pass their own test; all missing stays below)
  const bool up = best > INT32_MIN && best - floor0 > B.thr;
  if (__builtin_amdgcn_ballot_w64(up) == 0) return;
  B.thr = up ? best - floor0 : B.thr;
  B.browj = j0;
#pragma unroll
  for (int u = 0; u < 4; ++u) B.rv[u] = x[u];
}

// After 4 steps that hold column m for some lanes: its best cell in rows below n, or (ROW_N: the global optimum and a given
// end) its cell in row n.
template <bool FA, int R, bool ROW_N>
__device__ __forceinline__ void track_last_column(const KParams& P, const BandGroup<R>& G, int j0, int n, int m, int irow0,
                                                  BandBest<R>& B) {
  const bool here = j0 <= m && m <= j0 + 3;
  const unsigned long long b0 = __builtin_amdgcn_ballot_w64((m - j0) & 1), b1 = __builtin_amdgcn_ballot_w64((m - j0) & 2);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int v = mask_select(b1, mask_select(b0, G.v[3][r], G.v[2][r]), mask_select(b0, G.v[1][r], G.v[0][r]));
    const int i = irow0 + r + 1;
    const int sc = v - P.go - lane_zero<FA>() + (i + m) * P.ge;
    if (here && (ROW_N ? i == n : i < n && sc > B.bs)) {
      B.bs = sc;
      B.kj = i;
    }
  }
}

// The start of a band: a lane's row letters (kPad past the end), profile, column 0 and empty bests.
template <int MODE, int PROF, bool FA, int R>
__device__ __forceinline__ void band_start(const KParams& P, const uint32_t* sig2, const uint8_t* __restrict__ q, int n, bool flip, int irow0,
                                           int lane, uint32_t* __restrict__ lp, int (&prof)[R], BandLane<R>& L,
                                           BandBest<R>& B, bool& bad) {
  int rowc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = irow0 + r + 1;
    int c = kPad;
    if (i <= n) {
      c = q[i - 1];
      if (c >= P.alphabet) {
        bad = true;
        c = kPad;
      }
    }
    rowc[r] = c;
  }
  band_profile<PROF, R>(P, sig2, rowc, flip, prof, lp);
  // A lane also runs its columns before the first; global ones all hold column 0's value.
  const int jstart = MODE == ALN_GLOBAL ? 0 : -lane;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    L.h[r] = border_h<MODE, FA>(P, irow0 + r + 1, jstart);
    L.g[r] = lane_add<FA>(L.h[r], P.go, P.fgo);
    L.f[r] = lane_neg<FA>();
    for (int u = 0; u < 4; ++u) B.kv[u][r] = 0;
  }
  L.diag = border_h<MODE, FA>(P, irow0, jstart);
  L.bot_h = L.h[R - 1];
  L.bot_e = lane_neg<FA>();
  L.floor0 = lane_zero<FA>() - (irow0 + 1 + 1 - lane) * P.ge;
}

// The band's optimum in (score, i, j) order over the lane's rows, then across the wave.
template <int MODE, bool FA, int R>
__device__ __forceinline__ int4 band_optimum(const KParams& P, const BandBest<R>& B, int n,
                                             int m, bool flip, bool last_band, int irow0, bool bad, bool failed) {
  int bs = kNeg32, bi = 0, bjj = 0;
  const int rn = n - 1 - irow0;
  int br = -1, bj = -1;
  if (MODE == ALN_LOCAL) resolve_kept<R>(P, B, flip, br, bj);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = irow0 + r + 1;
    if (i > n) continue;
    const int sc = B.bs, jj = MODE == ALN_LOCAL ? bj : m;
    // row n's other columns are handled below
    const bool cand = MODE == ALN_LOCAL ? sc > 0 && r == br : i == B.kj;
    // a flipped pair's cell (i, jj) is the call's cell (jj, i)
    const int ci = flip ? jj : i, cj = flip ? i : jj;
    if (cand && better(sc, ci, cj, bs, bi, bjj)) {
      bs = sc;
      bi = ci;
      bjj = cj;
    }
  }
  if (MODE == ALN_SEMIGLOBAL && last_band && rn >= 0 && rn < R) {
    // row n: (n, 0) with H = 0 first, then its running maximum over j in column order
    int u = 3;
    if (B.rv[2] >= B.rv[3]) u = 2;
    if (B.rv[1] >= max(B.rv[2], B.rv[3])) u = 1;
    if (B.rv[0] >= max3i(B.rv[1], B.rv[2], B.rv[3])) u = 0;
    const int brow = B.thr - P.go + rn * P.ge, j = B.browj == INT32_MIN ? 0 : B.browj + u;
    const int ci = flip ? j : n, cj = flip ? n : j;
    if (better(brow, ci, cj, bs, bi, bjj)) {
      bs = brow;
      bi = ci;
      bjj = cj;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const int s2 = __shfl_xor(bs, o, 64), i2 = __shfl_xor(bi, o, 64), j2 = __shfl_xor(bjj, o, 64);
    if (better(s2, i2, j2, bs, bi, bjj)) {
      bs = s2;
      bi = i2;
      bjj = j2;
    }
  }
  return make_int4(bs, bi, bjj, (__any(bad) ? 1 : 0) | (failed ? 2 : 0));
}

// Fills the substitution scores sigma - 2 ge in LDS: the byte table, or for kProfTable the 32-bit table by (query
// letter, subject letter).
template <int PROF>
__device__ __forceinline__ void fill_table(const KParams& P, int32_t* tab, uint32_t* sig2) {
  if (PROF != kProfTable) {
    fill_score_bytes(P, sig2);
    return;
  }
  for (int k = threadIdx.x; k < kTab * kTab; k += blockDim.x) {
    const int a = k / kTab, b = k % kTab;
    tab[k] = (a >= P.alphabet || b >= P.alphabet) ? -kBig32 : (int32_t)P.sig[a * kMaxAlphabet + b] - 2 * P.ge;
  }
}

// The first ng of a block's groups of 4 steps.  A group's inputs are read from LDS while the group before runs (its
// letters one group earlier still where they lead to profile words), so that no group waits for LDS.
// AHEAD false: when the group starts, which leaves the waiting to the other waves of the SIMD and takes fewer registers.
template <int PROF, int R, int NG, bool AHEAD = true, typename Window, typename Rows, typename Run>
__device__ __forceinline__ void run_block(const Window& lett, const uint32_t* lp, int lane, int ng, Rows load_rows,
                                          Run run) {
  if constexpr (!AHEAD) {
    for (int g4 = 0; g4 < ng; ++g4) {
      BandIn<R> I;
      lett.get(lane, g4, I.vc);
      load_rows(g4, I);
      load_words<PROF, R>(lp, I);
      run(g4, I);
    }
    return;
  }
  BandIn<R> A, C;
  lett.get(lane, 0, A.vc);
  load_rows(0, A);
  if (lane_words(PROF)) lett.get(lane, 1, C.vc);
  load_words<PROF, R>(lp, A);
  for (int g4 = 0; g4 < ng; g4 += 2) {
    load_rows(g4 + 1, C);
    if (lane_words(PROF)) {
      load_words<PROF, R>(lp, C);
      lett.get(lane, g4 + 2, A.vc);
    } else {
      lett.get(lane, g4 + 1, C.vc);
    }
    run(g4, A);
    if (g4 + 1 >= ng) break;
    load_rows(g4 + 2, A);
    if (lane_words(PROF)) {
      load_words<PROF, R>(lp, A);
      lett.get(lane, g4 + 3, C.vc);
    } else {
      lett.get(lane, g4 + 2, A.vc);
    }
    run(g4 + 1, C);
  }
}

}  // namespace mialign
