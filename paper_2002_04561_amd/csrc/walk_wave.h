// Canonical traceback walk by a whole wave over 4-bit predecessor codes held in device memory.
//
// A cell's code is a nibble of its row group's 16-bit word, row r of the group at bits 4 (3 - r): bit 0 "H is not
// the diagonal", bit 1 "nor E", bit 2 "E extended a gap", bit 3 "F extended a gap"; a local cell with H = 0 has
// bits 1..0 = 10 (elsewhere bit 1 means nothing while bit 0 is clear).
//
// The walk of walk.h (the canonical rule: diagonal, then E, then F in the no-gap state; inside a gap
// the gap-open predecessor wins ties; local walks stop at a cell whose H is 0, semi-global ones on
// row 0 or column 0, global ones finish along row 0 or column 0), taken by one wave: the codes are
// read from an LDS window of kWalkCodes words loaded at the current cell (a window of 128 x 128 cells took 64 loads a lane and
// bound the walks of long pairs): along the diagonal, or, where the walk mostly goes up or left, a rectangle of many rows or of
// many columns (a 3500 x 300 global pair took 0.45 ms with the square one, 0.63 ms with diagonal ones alone, 0.34 ms so);
// diagonal runs are taken up to 64 cells at a time (lane t looks at cell (i - t, j - t), and the first
// lane whose cell is not a diagonal move, or lies outside the window or the codes, ends the run), and
// gap runs are taken the same way along their column or row.  Every lane runs the same walk and
// stores the same runs.
//
// The codes may cover only a segment of rows, r0 + 1 .. r0 + rows: the walk then stops when it
// reaches row r0 (in the no-gap state or inside a vertical gap), and a later call with the segment
// above continues it.  This is the linear-space traceback of AnySeq Sec. III-A: the segments are
// relaxed again one at a time from stored rows, so only one segment's codes are held at once.  They
// may also cover only the columns right of cb: the walk then stops when it reaches column cb, and a
// later call with the columns left of it continues.
#pragma once
#include "internal.h"

namespace mialign {

constexpr int kWalkCodes = 1024;  // row group words (of kWfR rows) in a traceback window
// Shapes: 32 row groups of 32 columns along the diagonal, the same as a rectangle, and 8 row groups of 128 columns.  The
// rectangles end at the cell that they were loaded at.
constexpr int kWalkLeft = 17;  // diagonal: columns left of the diagonal through the cell the window was loaded at
// A cell is in a diagonal window while its diagonal lies this far left or right of that cell's (the columns of a row group are
// placed for the group, so up to 3 columns are lost to either side).
constexpr int kWalkDiagLo = -(kWalkLeft - 3), kWalkDiagHi = 32 - 1 - kWalkLeft - 3;

template <int LOG_COLS, bool DIAG>
struct WalkShape {
  static constexpr int kLogCols = LOG_COLS;
  static constexpr bool kDiag = DIAG;
};

// A walk in progress.  Runs are stored last to first while walking; walk_finish reverses them.
struct WalkState {
  int32_t i, j;      // current cell (the begin cell once done)
  int32_t state;     // 0 = H, 1 = E (vertical gap, CIGAR I), 2 = F (horizontal gap, CIGAR D)
  int32_t done;      // the walk has reached the alignment's first cell
  uint32_t cur_op;   // the run being built (0xff: none yet)
  uint32_t cur_len;
  int64_t runs;      // runs stored so far
  int32_t stuck;     // the walk did not end within its bound of turns (never, for valid codes)
  int32_t pad_;
};

__device__ __forceinline__ void walk_start(WalkState& S, int i, int j) {
  S.i = i;
  S.j = j;
  S.state = 0;
  S.done = 0;
  S.cur_op = 0xffu;
  S.cur_len = 0;
  S.runs = 0;
  S.stuck = 0;
  S.pad_ = 0;
}

// Walks from S through the codes of rows rs + 1 .. and columns cb + 1 .. (row group g of the segment, whose rows start at
// r0 + 1, column c at codes[g * ld + c - 1]; rs >= r0).  Returns when the walk is done or has reached row rs > 0 or
// column cb > 0.
template <int MODE>
__device__ void walk_core(const uint16_t* __restrict__ codes, int64_t ld, int r0, int rs, int cb, WalkState& S,
                          uint16_t* __restrict__ win, int lane, uint32_t* __restrict__ cig, int64_t cap) {
  if (S.done) return;
  // Every lane holds the same walk state; saying so lets the compiler keep it in scalar registers
  // and branch on it with scalar branches.
  int i = __builtin_amdgcn_readfirstlane(S.i);
  int j = __builtin_amdgcn_readfirstlane(S.j);
  int state = __builtin_amdgcn_readfirstlane(S.state);
  uint32_t cur_op = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.cur_op);
  uint32_t cur_len = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.cur_len);
  // Runs collect in a register, lane r % 64 holding run r, and are stored 64 at a time: a store and its 64-bit bound for each run
  // lay on the walk's chain (1000 x 1000 global linear pair with CIGAR: 345 us, 339 so).  Those below first are stored already.
  uint32_t runs = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.runs), held = 0;  // (at most i + j + 1, below 2^32)
  const uint32_t first = runs;
  bool done = false;
  // H came from the diagonal: bits 1..0 clear, or, without local zeros, bit 0
  constexpr uint32_t kSrc = MODE == ALN_LOCAL ? 3u : 1u;
  auto store_runs = [&](uint32_t from, uint32_t to) __attribute__((always_inline)) {
    const uint32_t r = from + (uint32_t)lane;
    if (r >= first && r < to && r < cap) cig[r] = held;
  };
  auto push = [&](uint32_t op, uint32_t len) __attribute__((always_inline)) {
    if (op == cur_op) {
      cur_len += len;
      return;
    }
    if (cur_len) {
      held = (uint32_t)lane == (runs & 63u) ? (cur_len << 4) | cur_op : held;
      if ((++runs & 63u) == 0) store_runs(runs - 64, runs);
    }
    cur_op = op;
    cur_len = len;
  };
  int64_t turns = 2 * ((int64_t)i + j) + 64;

  // Loads a window at the walk's cell and walks until it leaves it.
  auto walk_window = [&](auto shape) __attribute__((always_inline)) {
    constexpr int LC = decltype(shape)::kLogCols, kCols = 1 << LC, kGroups = kWalkCodes >> LC;
    constexpr bool kDiag = decltype(shape)::kDiag;
    constexpr int kSlope = kDiag ? kWfR : 0, kLeft = kDiag ? kWalkLeft : kCols - 1;
    // Row group g0 - k's columns are c0 - kSlope k - kLeft ...  The walk only moves up and left, so a later cell is inside the
    // window while it lies at or below row ilo and at or right of column jlo (the first that the walk may take) and, in a
    // diagonal window, on a diagonal within kWalkDiagLo .. kWalkDiagHi of the first cell's.
    const int g0 = (i - r0 - 1) / kWfR, c0 = j, i0 = i;
    const int ilo = max(rs + 1, r0 + (g0 - kGroups + 1) * kWfR + 1);
    const int jlo = kDiag ? cb + 1 : max(cb + 1, c0 - kLeft);
    {
      // Every load of the window is issued before the first LDS write, so the reload costs one memory
      // latency rather than one per code.  A window cell outside the segment (row group < 0) or the columns
      // loads the in-bounds cell (g0, c0) instead; the walk never reads it.  The loads carry no branches, so all
      // of them stay in flight together.
      constexpr int kPer = kWalkCodes / 64;
      uint32_t v[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int w = lane + 64 * u;
        const int k = w >> LC, gg = g0 - k, cc = c0 - kSlope * k - kLeft + (w & (kCols - 1));
        const bool ok = gg >= 0 && cc >= 1 && cc <= ld;
        v[u] = codes[(size_t)(ok ? gg : g0) * (size_t)ld + (size_t)((ok ? cc : c0) - 1)];
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u) win[lane + 64 * u] = (uint16_t)v[u];
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // the window is in LDS before it is read
    }
    // the code of a cell inside the window
    auto code = [&](int ii, int jj) __attribute__((always_inline)) -> uint32_t {
      const unsigned r = (unsigned)(ii - r0 - 1);
      const int k = g0 - (int)(r / kWfR);
      const uint32_t w = win[k * kCols + (jj - c0 + kSlope * k + kLeft)];
      return (w >> (4 * (kWfR - 1 - r % kWfR))) & 15u;
    };
    for (; turns > 0; --turns) {
      if (state == 0) {
        const int off = (j - c0) - (i - i0);
        // (rows up to rs and columns up to cb are outside the window)
        if (i < ilo || j < jlo || (kDiag && (off < kWalkDiagLo || off > kWalkDiagHi))) return;
        // lanes t <= lim look at cells inside the window; the others read (i, j) and count as a
        // non-diagonal code, which ends the run
        const int lim = min(i - ilo, j - jlo);
        const bool in = lane <= lim;
        const int t = in ? lane : 0;
        const uint32_t ct = code(i - t, j - t);
        const uint32_t pc = in ? ct : 3u;
        const unsigned long long ends = __builtin_amdgcn_ballot_w64((pc & kSrc) != 0u);
        const int k = ends ? __builtin_ctzll(ends) : 64;
        if (k > 0) {
          push(ALN_CIGAR_M, (uint32_t)k);
          i -= k;
          j -= k;
        }
        if (k == 64 || k > lim) continue;
        // lane k looked at the cell that ends the run, which the window holds; its code also gives the first gap
        // step, taken below without reading the cell again
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)pc, k);
        if (MODE == ALN_LOCAL && (c & 3u) == 2u) {
          done = true;  // H = 0
          return;
        }
        const bool up = !(c & 2u);
        push(up ? ALN_CIGAR_I : ALN_CIGAR_D, 1);
        state = up ? ((c & 4u) && i > 1 ? 1 : 0) : ((c & 8u) && j > 1 ? 2 : 0);
        i -= up ? 1 : 0;
        j -= up ? 0 : 1;
      } else {
        // A gap run, up to 64 steps at a time: lane t looks at the t-th cell of the run.  The run goes
        // on through a cell whose extension bit is set and which is not in row (column) 1; the first
        // cell that ends it is stepped through and returns the walk to H, unless it lies outside the
        // window, where the walk stops short of it and reloads.
        const int off = (j - c0) - (i - i0);
        if (i < ilo || j < jlo || (kDiag && (off < kWalkDiagLo || off > kWalkDiagHi))) return;
        const bool vert = state == 1;
        // lanes t <= lim look at cells inside the window
        const int lim = vert ? (kDiag ? min(i - ilo, kWalkDiagHi - off) : i - ilo)
                             : (kDiag ? min(j - jlo, off - kWalkDiagLo) : j - jlo);
        const bool in = lane <= lim;
        const int t = in ? lane : 0;
        const int ii = vert ? i - t : i, jj = vert ? j : j - t;
        const uint32_t pc = code(ii, jj);
        const bool more = in && (pc & (vert ? 4u : 8u)) != 0u && (vert ? ii : jj) > 1;
        const unsigned long long last = __builtin_amdgcn_ballot_w64(!more);
        const int k = last ? __builtin_ctzll(last) : 64;
        const bool ends = k < 64 && k <= lim;
        const int steps = k + (ends ? 1 : 0);
        push(vert ? ALN_CIGAR_I : ALN_CIGAR_D, (uint32_t)steps);
        i -= vert ? steps : 0;
        j -= vert ? 0 : steps;
        if (ends) state = 0;
      }
    }
  };
  int pi = i, pj = j;  // the cell the last window was loaded at
  while (turns > 0 && !done) {
    if (state == 0 && (i == 0 || j == 0)) {
      if (MODE == ALN_GLOBAL) {
        if (j > 0) push(ALN_CIGAR_D, (uint32_t)j);
        if (i > 0) push(ALN_CIGAR_I, (uint32_t)i);
        i = 0;
        j = 0;
      }
      done = true;
      break;
    }
    if (state != 2 && i == rs) break;  // the rows above hold this cell, or the vertical gap goes on there
    if (cb > 0 && j == cb) break;      // the columns left of cb hold it, or the gap goes on in (or ends at) them
    // a gap that has left its window, or a walk that went twice as far up as left (or left as up) through the last
    const int di = pi - i, dj = pj - j;
    pi = i;
    pj = j;
    if (state ? state == 1 : di > 2 * dj)
      walk_window(WalkShape<5, false>{});
    else if (state ? state == 2 : dj > 2 * di)
      walk_window(WalkShape<7, false>{});
    else
      walk_window(WalkShape<5, true>{});
  }
  store_runs(runs & ~63u, runs);
  if (turns <= 0) {
    S.stuck = 1;
    done = true;
  }
  S.i = i;
  S.j = j;
  S.state = state;
  S.done = done ? 1 : 0;
  S.cur_op = cur_op;
  S.cur_len = cur_len;
  S.runs = runs;
}

// Ends a walk: stores the last run and reverses the runs (last to first while walking) with the whole
// wave.  Lane l swaps the pairs (a, runs-1-a) with a = l, l+64, ...: no two lanes touch the same run.  Run r
// was stored by lane r % 64, so a lane loads other lanes' stores: the wait before the swap completes them.
// Returns the number of runs.
__device__ inline int64_t walk_finish(WalkState& S, int lane, uint32_t* __restrict__ cig, int64_t cap) {
  int64_t runs = S.runs;
  if (S.cur_len) {
    if (runs < cap) cig[runs] = (S.cur_len << 4) | S.cur_op;
    ++runs;
  }
  S.cur_len = 0;
  S.runs = runs;
  if (runs <= cap) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int64_t half = runs / 2;
    for (int64_t a = lane; a < half; a += 64) {
      const int64_t b = runs - 1 - a;
      const uint32_t x = cig[a], y = cig[b];
      cig[a] = y;
      cig[b] = x;
    }
  }
  return runs;
}

}  // namespace mialign
