// The cell recurrence of the band wavefronts (the grouped and per-band engines of wf_i32.hip and the
// traceback tiles of tb_tiles.hip): four steps of a lane's rows.
//
// Every value carries the bias (i + j) * |ge|: H~(i,j) = H(i,j) - (i + j) * ge, and likewise E and F.  Then
// extending either gap costs nothing, and both gaps open from the same sum:
//   g(i,j)  = H~(i,j) + go
//   E~(i,j) = max(E~(i-1,j), g(i-1,j))                  Eq. (4)
//   F~(i,j) = max(F~(i,j-1), g(i,j-1))                  Eq. (5)
//   H~(i,j) = max(H~(i-1,j-1) + sigma - 2 ge, E~, F~ [, the floor: H = 0])   Eq. (1)
// -- with affine gaps one addition, one dot product that also picks the substitution score, and three maxima per cell; with
// linear ones (go = 0, g = H~) an extract, an addition and the maximum of three.
//
// What bounds it: VALU issue.  Measured on gfx950 (independent chains, 4 and more waves per SIMD), a
// wave64 max, max3, bit-field extract, byte permute, alignbit, dot4 or DPP move takes 4.2 cycles; an integer
// add takes 2.4 alone but 3.9 next to those; and an fp32 add takes 2.3 and runs beside another wave's max,
// max3, alignbit or extract (4.5 cycles for the two).  So:
//   - v_dot4_i32_i8 with a one-hot operand picks a signed byte of the profile and adds it to the diagonal
//     (4.2 cycles; extract and add took 4.2 + 3.9);
//   - with FA the lanes hold every value v as the bits of the float 2^23 + 2^20 + v, in 2^23 .. 2^24, where
//     one float step is one integer step: integer maxima, comparisons and dot4 work on the bits, and adding
//     a constant is an exact fp32 add, which the SIMD issues beside the maxima.  The host allows FA when
//     every value provably stays in that range (band_fits_fa); otherwise the same code adds integers.
// With these cells and the optima tracked in groups (band_wave.h) 65,536 local affine protein pairs of 64..16384 letters took
// 118 ms and 8.4 VALU lane-operations a cell, where a row bias alone took 160 ms and 11.8.
#pragma once
#include "internal.h"

namespace mialign {

// Where a band's substitution scores sigma(row letter, column letter) - 2 ge come from:
//   kProfTable  a 32-bit LDS table indexed by both letters (any score range);
//   kProfReg    alphabets of up to 4 letters: one register per row holds the scores of the row's
//               letter against the 4 letters as signed bytes; a column letter is the one-hot byte 1 << 8c;
//   kProfRegBits the same registers, a column letter as the bit offset 8c, for an extract and an add;
//   kProfLane   alphabets of up to 32 letters: per letter, every lane keeps the scores of 4 rows as 4
//               signed bytes in one LDS word, so a step reads one word per 4 rows;
//   kProfRegLow, kProfLaneLow  the two for scores past a byte: the bytes hold sigma - 2 ge - sig_off, and a cell adds
//               sig_off back.  The one addition more is dear where cells fill the SIMD (1500 linear-gap protein pairs of
//               2000..6000 3.28 ms without and 3.71 with), and the table dearer yet: extend -70, 4 letters, local,
//               30000 x 30000 8.25 ms from the table and 5.34 so, 3000 of 64..2000 2.56 and 1.64.
// The byte forms need every one of their bytes in -127..127 (-128 marks rows past the end).
constexpr int kProfTable = 0, kProfReg = 1, kProfLane = 2, kProfRegBits = 3, kProfRegLow = 4, kProfLaneLow = 5;
constexpr bool reg_bits(int prof) { return prof == kProfRegBits || prof == kProfRegLow; }  // column letters as bit offsets
constexpr bool lane_words(int prof) { return prof == kProfLane || prof == kProfLaneLow; }
constexpr uint32_t kPadWord = 0x80808080u;  // four rows past the end, or the letter past a subject's end

constexpr int kFaBits = 0x4B000000;  // the float 2^23
// the lane value that stands for 0, and one that every value exceeds
template <bool FA>
__device__ __forceinline__ constexpr int lane_zero() {
  return FA ? kFaBits + (1 << 20) : 0;
}
template <bool FA>
__device__ __forceinline__ constexpr int lane_neg() {
  return FA ? kFaBits : kNeg32;
}
// v + k, k given both as an integer and as the same float
template <bool FA>
__device__ __forceinline__ int lane_add(int v, int k, float kf) {
  if constexpr (FA) return __builtin_bit_cast(int, __builtin_bit_cast(float, v) + kf);
  int r = v + k;
  asm("" : "+v"(r));  // keeps the compiler from rearranging sums: it takes 50 registers more when it does
  return r;
}
// bit 31: a < b
template <bool FA>
__device__ __forceinline__ uint32_t lane_lt(int a, int b) {
  if constexpr (FA) return __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, a) - __builtin_bit_cast(float, b));
  return (uint32_t)(a - b);
}
__device__ __forceinline__ int max3i(int a, int b, int c) { return max(max(a, b), c); }

// A lane's rows of a band: H~, g and F~ of the column last relaxed, H~ of the row above at that column
// (the next diagonal), and the bottom row's H~ and E~, which the lane below takes at the next step.
template <int R>
struct BandLane {
  int h[R], g[R], f[R];
  int diag, bot_h, bot_e;
  int floor0;  // local and semi-global: the lane value of H = 0 at the first row and the column of the next step
};

// H~(i, j) of a cell on row 0 or column 0
template <int MODE, bool FA>
__device__ __forceinline__ int border_h(const KParams& P, int i, int j) {
  if (MODE == ALN_GLOBAL) return lane_zero<FA>() + (i + j > 0 ? P.go : 0);
  return lane_zero<FA>() - (i + j) * P.ge;
}

// The traceback word of a column: a nibble per row, row r at bits 4 (R - 1 - r); bit 0 "not the diagonal",
// bit 1 "neither the diagonal nor E" (non-local: "not E"), bit 2 "E extended", bit 3 "F extended".  Local cells
// with H = 0 have bits 1..0 = 10.  Each flag is the sign of a difference, shifted in by v_alignbit: one issue
// slot a flag beside an fp32 subtraction; comparing and selecting took two to three.
__device__ __forceinline__ uint32_t push_flag(uint32_t acc, uint32_t sign) {
  return __builtin_amdgcn_alignbit(acc, sign, 31);
}

// How a group of steps treats columns outside 1..m.  Local cells there need nothing: left of the matrix they hold the floor,
// H = 0, which is column 0's value, and right of it they are below real cells.  In the other modes cells right of the matrix are
// never used (column m is kept as it passes), and left of it they are kept at the border value by a floor of their own in the
// first groups (kGroupStart).  Masking the updates instead took a branch a step, which kept the steps from overlapping, in the
// 33 edge groups of a band (100003 reads of 100..250, scores: 2.26 ms, 2.14 so).
// kGroupChecked masks them: the traceback's tiles start from any column.
enum { kGroupInside = 0, kGroupStart = 1, kGroupChecked = 2 };

// One column of a lane's rows.  in_h, in_e: H~ and E~ of the row above; in_c: the column letter (as the
// profile kind wants it); pw: kProfLane, its words; fl[r]: the floor of row r (with FLOOR).  With TB the column's R nibbles
// are shifted into acc; otherwise a local affine cell folds its floor into E, which leaves H as it is: the floor
// is one of H's terms anyway, and an E raised to row i's floor stays below the floor of every row beneath it.
template <int MODE, bool AFFINE, int PROF, bool TB, bool FA, int R, bool FLOOR>
__device__ __forceinline__ void band_column(const KParams& P, const int32_t* tab, const int (&prof)[R],
                                            const int (&pw)[(R + 3) / 4], int in_c, int in_h, int in_e,
                                            const int* fl, BandLane<R>& L, uint32_t& acc) {
  int gup = AFFINE ? lane_add<FA>(in_h, P.go, P.fgo) : in_h;
  int e = in_e, hd = L.diag;
  L.diag = in_h;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int d;
    // Linear gaps add nothing else to a cell: a step waits for its chain of maxima, and the extract and add that the chain does not wait
    // for beat the dot product's latency (30000 x 30000 proteins 5.17 and 4.64 ms, 3000 of 64..2000 semi-global 1.38 and 1.01).
    if constexpr (PROF == kProfRegBits)
      d = hd + __builtin_amdgcn_sbfe(prof[r], in_c, 8);
    else if constexpr (PROF == kProfRegLow)
      d = hd + P.sig_off + __builtin_amdgcn_sbfe(prof[r], in_c, 8);
    else if constexpr (PROF == kProfLaneLow)
      d = hd + P.sig_off + __builtin_amdgcn_sbfe(pw[r / 4], 8 * (r & 3), 8);
    else if constexpr (PROF == kProfLane && !AFFINE)
      d = hd + __builtin_amdgcn_sbfe(pw[r / 4], 8 * (r & 3), 8);
    else if constexpr (PROF == kProfReg)
      d = __builtin_amdgcn_sdot4(prof[r], in_c, hd, false);
    else if constexpr (PROF == kProfLane)
      d = __builtin_amdgcn_sdot4(pw[r / 4], 1 << (8 * (r & 3)), hd, false);
    else
      d = hd + tab[prof[r] + in_c];
    // (a pad column left of the matrix must not rise above the border value by the lowered bytes' offset)
    if (PROF == kProfRegLow && MODE == ALN_GLOBAL && FLOOR) d = in_c == 31 ? hd : d;
    const int gl = AFFINE ? L.g[r] : L.h[r];
    constexpr bool kFold = FLOOR && AFFINE && !TB;
    if (AFFINE)
      e = kFold ? max3i(e, gup, fl[r]) : max(e, gup);
    else
      e = gup;
    const int f = AFFINE ? max(L.f[r], gl) : gl;
    const int dm = FLOOR && !kFold ? max(d, fl[r]) : d;
    const int h = max3i(dm, e, f);
    if (TB) {
      if (AFFINE) {
        acc = push_flag(acc, lane_lt<FA>(gl, f));
        acc = push_flag(acc, lane_lt<FA>(gup, e));
      } else {
        acc <<= 2;
      }
      if (MODE == ALN_LOCAL)
        acc = push_flag(acc, lane_lt<FA>(max(d, e), max(h, fl[r] + 1)));
      else
        acc = push_flag(acc, lane_lt<FA>(e, h));
      acc = push_flag(acc, lane_lt<FA>(dm, h));
    }
    hd = L.h[r];
    L.h[r] = h;
    if (AFFINE) {
      L.f[r] = f;
      L.g[r] = lane_add<FA>(h, P.go, P.fgo);
    }
    gup = AFFINE ? L.g[r] : h;
  }
  L.bot_h = L.h[R - 1];
  L.bot_e = e;
}

// What a group of 4 steps leaves for its caller.
template <int R>
struct BandGroup {
  int v[4][R];       // every cell's g with affine gaps, its H~ with linear ones (where g = H~)
  int oh[4], oe[4];  // the bottom row: H~ and E~
  uint32_t cw[4];    // TB: the column's nibbles in the low bits (and the column before above them)
};

// The inputs of 4 steps: vh, ve are the wave's top row there (lane 0 takes them; the others take the lane above's
// bottom row), vc the lane's column letters, pw (kProfLane) their profile words.
template <int R>
struct BandIn {
  int vh[4], ve[4], vc[4];
  int pw[4][(R + 3) / 4];
};
template <int PROF, int R>
__device__ __forceinline__ void load_words(const uint32_t* lp, BandIn<R>& I) {
  if constexpr (lane_words(PROF)) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < R / 4; ++k)
        I.pw[u][k] = (int)*reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lp) + I.vc[u] + 256 * k);
  }
}

// Four steps.  Lane l of the wave is at columns j0 .. j0 + 3.  after(u) runs after step u.
template <int MODE, bool AFFINE, int PROF, bool TB, bool FA, int R, int EDGE, typename After>
__device__ __forceinline__ void band_group(const KParams& P, const int32_t* tab, const int (&prof)[R],
                                           const BandIn<R>& I, int j0, int m, BandLane<R>& L, BandGroup<R>& G,
                                           After after) {
  constexpr bool kStart = EDGE == kGroupStart && MODE != ALN_LOCAL;
  constexpr bool kFloor = MODE == ALN_LOCAL || kStart;
  int fl[R + 3];
#pragma unroll
  for (int k = 0; k < R + 3; ++k) {
    fl[k] = 0;
    if (MODE == ALN_LOCAL) fl[k] = k ? lane_add<FA>(L.floor0, -k * P.ge, P.fc[k]) : L.floor0;
  }
  uint32_t acc = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int in_h = __builtin_amdgcn_update_dpp(I.vh[u], L.bot_h, 0x138, 0xf, 0xf, false);  // wave_shr:1
    const int in_e = AFFINE ? __builtin_amdgcn_update_dpp(I.ve[u], L.bot_e, 0x138, 0xf, 0xf, false) : 0;
    if constexpr (kStart) {
      // the border value of the lane's first row left of column 1, and no floor from there on
      const int level = MODE == ALN_GLOBAL ? lane_zero<FA>() + P.go
                        : u                ? lane_add<FA>(L.floor0, -u * P.ge, P.fc[u])
                                           : L.floor0;
      int fs[R];
      fs[0] = j0 + u <= 0 ? level : lane_neg<FA>();
#pragma unroll
      for (int r = 1; r < R; ++r)
        fs[r] = MODE == ALN_GLOBAL ? fs[0] : lane_add<FA>(fs[0], -r * P.ge, P.fc[r]);
      band_column<MODE, AFFINE, PROF, TB, FA, R, true>(P, tab, prof, I.pw[u], I.vc[u], in_h, in_e, fs, L, acc);
    } else if (EDGE != kGroupChecked || (j0 + u >= 1 && j0 + u <= m)) {
      band_column<MODE, AFFINE, PROF, TB, FA, R, kFloor>(P, tab, prof, I.pw[u], I.vc[u], in_h, in_e, fl + u, L, acc);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) G.v[u][r] = AFFINE ? L.g[r] : L.h[r];
    G.oh[u] = L.bot_h;
    G.oe[u] = L.bot_e;
    G.cw[u] = acc;
    after(u);
  }
  if (MODE != ALN_GLOBAL) L.floor0 = lane_add<FA>(L.floor0, -4 * P.ge, P.fc[4]);
}

// The traceback words of a group's 4 columns, first column first.
template <int R>
__device__ __forceinline__ uint2 group_words(const BandGroup<R>& G) {
  return make_uint2(__builtin_amdgcn_alignbit(G.cw[1], G.cw[1], 16), __builtin_amdgcn_alignbit(G.cw[3], G.cw[3], 16));
}

// Stores a group's traceback words.  Groups inside the matrix write 4 columns at once (8 bytes at an address
// of 2-byte alignment, which global stores allow); at the edges each valid column is stored on its own.
struct __attribute__((packed, aligned(2))) Words4 {
  uint32_t a, b;
};
template <int R>
__device__ __forceinline__ void store_codes(const BandGroup<R>& G, uint16_t* __restrict__ codes, int j0, int m,
                                            bool inside) {
  if (inside) {
    const uint2 w = group_words<R>(G);
    Words4 v;
    v.a = w.x;
    v.b = w.y;
    *reinterpret_cast<Words4*>(codes + (j0 - 1)) = v;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j0 + u >= 1 && j0 + u <= m) codes[j0 + u - 1] = (uint16_t)G.cw[u];
  }
}

// Profile entries of a lane's R rows (letters rowc, kPad past the end): registers, or the lane's words of
// lp ([letter][64-lane block of 4 rows], the pad letter last).  flip: the rows are the subject's.  sig2: the LDS copy
// of the byte table KParams::sig2.
constexpr int kScoreWords = 2 * kMaxAlphabet * kMaxAlphabet / 4;
__device__ __forceinline__ void fill_score_bytes(const KParams& P, uint32_t* sig2) {
  for (int k = threadIdx.x; k < kScoreWords; k += blockDim.x) sig2[k] = reinterpret_cast<const uint32_t*>(P.sig2)[k];
}
template <int PROF, int R>
__device__ __forceinline__ void band_profile(const KParams& P, const uint32_t* sig2, const int (&rowc)[R], bool flip,
                                             int (&prof)[R], uint32_t* __restrict__ lp) {
  // kMaxAlphabet bytes per row letter, by query letter first or by subject letter
  const uint32_t* rows = sig2 + (flip ? kMaxAlphabet * 8 : 0);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (PROF == kProfReg || reg_bits(PROF))
      prof[r] = (int)(rowc[r] < kMaxAlphabet ? rows[rowc[r] * 8] : kPadWord);
    else if (PROF == kProfTable)
      prof[r] = flip ? rowc[r] : rowc[r] * kTab;  // the table is indexed [query letter][subject letter]
    else
      prof[r] = 0;
  }
  if constexpr (lane_words(PROF)) {
    constexpr int NW = R / 4;
    for (int a = 0; a < P.alphabet; a += 4) {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        uint32_t w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = rowc[4 * k + r] < kMaxAlphabet ? rows[rowc[4 * k + r] * 8 + a / 4] : kPadWord;
        // 4 x 4 bytes, rows to letters
        const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
        const uint32_t hi01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
        const uint32_t hi23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
        const uint32_t t[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u),
                               __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                               __builtin_amdgcn_perm(hi23, hi01, 0x05040100u),
                               __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (a + b < P.alphabet) lp[((a + b) * NW + k) * 64] = t[b];
      }
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) lp[(P.alphabet * NW + k) * 64] = kPadWord;
  }
}

// A subject letter as the profile kind wants it; col < 1 or past the end (c < 0) gives the pad letter, whose
// score is at most 2 ge, or at most -1 of the lowered bytes: a cell of a pad column is below a real cell.
template <int PROF, int R>
__device__ __forceinline__ int letter_index(const KParams& P, int c, bool flip, bool& bad) {
  if (c >= P.alphabet) {
    bad = true;
    c = -1;
  }
  if (PROF == kProfReg) return c < 0 ? 0 : 1 << (8 * c);
  if (reg_bits(PROF)) return c < 0 ? 31 : 8 * c;  // (the extract at bit 31 gives 0 or -1)
  if (lane_words(PROF)) return (c < 0 ? P.alphabet : c) * 256 * (R / 4);  // bytes
  return (c < 0 ? kPad : c) * (flip ? kTab : 1);
}

}  // namespace mialign
