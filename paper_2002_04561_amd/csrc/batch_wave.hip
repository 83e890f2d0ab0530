// One wave per pair: traceback batches too short to fill the one-pair-per-lane kernels, and aln_traceback.
//
// A lane of batch_i16.hip takes a whole pair, so a batch takes at least as long as its largest pair on one lane: 4.5 ms
// for 400 reads of 100..250 letters against windows 64 longer, and 8.1 for 262,144 of them.  Here a wave relaxes its pair
// band by band (256 rows: 64 lanes x 4) with the recurrence of band.h, in 32-bit lanes, keeps the bottom row of a band in a
// row buffer of its own for the next, and walks the codes back with the whole wave (walk_wave.h).  Bound by VALU issue:
// a read's band takes (m + 64) steps of about 55 instructions, about 46 % of its lane-steps padding (256 rows for 175, m + 64 steps for m).
// Pairs come in the planner's order, largest first, and the waves take them in turn.
#include "band.h"
#include "band_wave.h"
#include "internal.h"
#include "walk_wave.h"

#include <algorithm>
#include <type_traits>

namespace mialign {
namespace {

constexpr int kPWavesPerBlock = 4;
// Three waves a SIMD (168 registers each): four, with 128, spilled 9 to 180 of them (20011 reads of 100..250 traced back from
// their ends 732 us, 722 so; 400 such reads with CIGARs 109 us, 104 so).  At three the semi-global reads and all linear gaps fit;
// the local affine kernels still spill 19 to 37, and two semi-global ones with the table 13 and 15.
constexpr int kPWavesPerCU = 12;
constexpr int kPBand = 64 * kWfR;

// LDS of one wave: while it relaxes, the stage of top-row inputs and outputs (H~ and E~ of 64 columns), the letter window and
// the profile words; then the window of its walk.
constexpr int kPStageBytes = 2 * 64 * 4;
constexpr int kPLettersBytes = (int)((sizeof(LetterWindow<64>) + 15) / 16 * 16);
__host__ __device__ constexpr int pair_lds_bytes(int alphabet, bool lane_profile) {
  const int relax = kPStageBytes + kPLettersBytes + (lane_profile ? (alphabet + 1) * 256 : 0);
  const int walk = kWalkCodes * 2;
  return relax > walk ? relax : walk;
}

// Relaxes a pair (n, m > 0) and stores its codes ([row group][column]); returns its optimum (score, i, j), or with FIXED the
// score of cell (n, m) alone.
template <int MODE, bool AFFINE, int PROF, bool FA, bool FIXED>
__device__ __forceinline__ int4 relax_pair(const KParams& P, const int32_t* tab, const uint32_t* sig2, char* lds,
                                           const uint8_t* __restrict__ q, int n, const uint8_t* __restrict__ s, int m,
                                           int lane, int2* __restrict__ row, uint16_t* __restrict__ codes0, bool& bad) {
  constexpr int R = kWfR, BLK = 64;
  int* st_h = reinterpret_cast<int*>(lds);
  int* st_e = st_h + 64;
  LetterWindow<64>& lett = *reinterpret_cast<LetterWindow<64>*>(lds + kPStageBytes);
  uint32_t* lp = reinterpret_cast<uint32_t*>(lds + kPStageBytes + kPLettersBytes) + lane;
  const int nb = (n + kPBand - 1) / kPBand;
  const int steps = m + 64;
  int4 best = make_int4(kNeg32, 0, 0, 0);
  for (int b = 0; b < nb; ++b) {
    const int i0 = b * kPBand, irow0 = i0 + lane * R;
    int prof[R];
    BandLane<R> L;
    BandBest<R> B;
    band_start<MODE, PROF, FA, R>(P, sig2, q, n, false, irow0, lane, lp, prof, L, B, bad);
    uint16_t* __restrict__ codes = codes0 + (size_t)(b * 64 + lane) * (size_t)m;
    const bool last_band = b == nb - 1;
    if (MODE == ALN_SEMIGLOBAL && last_band) last_row_start<R>(P, n - 1 - irow0, B);
    int c_next = 1 + lane <= m ? (int)s[lane] : -1;
    int c_idx = letter_index<PROF, R>(P, -1, false, bad);
    lett.clear_tail(lane);
    for (int tb = 0; tb < steps; tb += BLK) {
      const int col_in = tb + 1 + lane;
      const int c_old = c_idx;
      c_idx = letter_index<PROF, R>(P, c_next, false, bad);
      lett.put(lane, c_old, c_idx);
      c_next = col_in + BLK <= m ? (int)s[col_in + BLK - 1] : -1;
      int32_t th = lane_neg<FA>(), te = lane_neg<FA>();
      if (col_in <= m) {
        if (b == 0) {
          th = border_h<MODE, FA>(P, 0, col_in);
        } else {
          const int2 v = row[col_in];
          th = v.x;
          te = v.y;
        }
      }
      if (MODE == ALN_LOCAL && !FIXED)
        B.floor = raise_local_floor(B.bs, col_in <= m ? th - lane_zero<FA>() + (i0 + col_in) * P.ge : 0);
      st_h[lane] = th;
      st_e[lane] = te;
      auto load_rows = [&](int g4, BandIn<R>& I) __attribute__((always_inline)) {
        const int4 h4 = reinterpret_cast<const int4*>(st_h)[g4 & 15];
        const int4 e4 = reinterpret_cast<const int4*>(st_e)[g4 & 15];
        I.vh[0] = h4.x, I.vh[1] = h4.y, I.vh[2] = h4.z, I.vh[3] = h4.w;
        I.ve[0] = e4.x, I.ve[1] = e4.y, I.ve[2] = e4.z, I.ve[3] = e4.w;
      };
      auto run = [&](int g4, const BandIn<R>& I) __attribute__((always_inline)) {
        const int t0 = tb + 4 * g4;
        const int j0 = t0 - lane + 1;
        const int ph = L.bot_h, pe = L.bot_e, floor0 = L.floor0;
        BandGroup<R> G;
        const bool inside = t0 >= 63 && t0 + 3 < m;
        if (MODE == ALN_LOCAL || t0 >= 63)
          band_group<MODE, AFFINE, PROF, true, FA, R, kGroupInside>(P, tab, prof, I, j0, m, L, G, [](int) {});
        else
          band_group<MODE, AFFINE, PROF, true, FA, R, kGroupStart>(P, tab, prof, I, j0, m, L, G, [](int) {});
        if ((MODE != ALN_LOCAL || FIXED) && t0 + 4 >= m)
          track_last_column<FA, R, MODE == ALN_GLOBAL || FIXED>(P, G, j0, n, m, irow0, B);
        if (irow0 < n) store_codes<R>(G, codes, j0, m, inside);  // row groups past n have no room
        if constexpr (!FIXED) {
          if constexpr (MODE == ALN_LOCAL) track_local<AFFINE, R>(P, L, G, floor0, j0, false, B);
          if (MODE == ALN_SEMIGLOBAL && last_band) track_last_row<AFFINE, R>(P, L, G, floor0, m, n - 1 - i0, j0, B);
        }
        if (lane == 63) {
          reinterpret_cast<int4*>(st_h)[g4] = make_int4(ph, G.oh[0], G.oh[1], G.oh[2]);
          reinterpret_cast<int4*>(st_e)[g4] = make_int4(pe, G.oe[0], G.oe[1], G.oe[2]);
        }
      };
      run_block<PROF, R, BLK / 4>(lett, lp, lane, min(BLK / 4, (steps - tb + 3) / 4), load_rows, run);
      // slot u now holds lane 63's column tb + u - 63, whose entry of the row above has been read
      if (!last_band) {
        const int col_out = tb + lane - 63;
        if (col_out >= 1 && col_out <= m) row[col_out] = make_int2(st_h[lane], st_e[lane]);
      }
    }
    // the row buffer's stores are complete before the next band's lanes read other lanes' columns
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (FIXED) {
      if (last_band) {
        best = make_int4(__builtin_amdgcn_readlane(B.bs, (n - 1 - i0) / R), n, m, 0);
      }
    } else {
      const int4 o = band_optimum<MODE, FA, R>(P, B, n, m, false, last_band, irow0, false, false);
      if (better(o.x, o.y, o.z, best.x, best.y, best.z)) best = o;
    }
  }
  return best;
}

// FIXED: trace back from the end cell a forward pass found (fwd[p].q_end, fwd[p].s_end); the pair is relaxed only up to that
// cell, whose H must equal fwd[p].score.
template <int MODE, bool AFFINE, int PROF, bool FA, bool FIXED>
__global__ __launch_bounds__(64 * kPWavesPerBlock, kPWavesPerCU / 4) void batch_wave_kernel(const KParams P, const WaveArgs A, int n_waves,
                                                                             size_t wave_bytes, size_t row_bytes) {
  // FIXED falls back to the 32-bit table, whose pad letter no alignment takes, where a letter is invalid: its H must be
  // the one of aln_traceback's other kernel
  constexpr bool kTable = PROF == kProfTable || FIXED;
  __shared__ int32_t tab[kTable ? kTab * kTab : 1];
  __shared__ uint32_t sig2[PROF == kProfTable ? 1 : kScoreWords];
  extern __shared__ char smem[];
  if constexpr (kTable) fill_table<kProfTable>(P, tab, nullptr);
  if constexpr (PROF != kProfTable) fill_score_bytes(P, sig2);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  char* lds = smem + wib * pair_lds_bytes(P.alphabet, PROF == kProfLane);
  const int64_t wave = (int64_t)blockIdx.x * kPWavesPerBlock + wib;
  if (wave >= n_waves) return;
  char* slab = static_cast<char*>(A.ws) + wave * wave_bytes;
  int2* row = reinterpret_cast<int2*>(slab);
  uint16_t* codes = reinterpret_cast<uint16_t*>(slab + row_bytes);
  int64_t count = A.idx ? (int64_t)*A.idx_count : A.n_pairs;
  if (FIXED && A.work) {
    static_assert(kWorkSlots == 64, "a slot per lane");
    const PairWork w = wave_work(A.work[lane]);
    const bool waves = (double)w.steps * A.step_ns <= (double)w.cells * A.cell_ns;
    if (wave == 0 && lane == 0) *A.lane_count = waves ? 0 : (int)A.n_pairs;
    if (!waves) count = 0;
  }
  if (A.zero && wave == 0 && lane < A.n_zero) A.zero[lane] = 0;
  for (int64_t slot = wave; slot < count; slot += n_waves) {
    const int64_t p = A.idx ? (int64_t)A.idx[slot] : slot;
    const int64_t qb = A.q_off[p], sb = A.s_off[p];
    const int64_t nn = A.q_off[p + 1] - qb, mm = A.s_off[p + 1] - sb;
    int n = 0, m = 0;
    uint32_t flags = 0;
    aln_result_t fw{};
    // (the list may hold a longer pair than the slabs: one that found no room in an arena sized from understated totals)
    if (nn > A.max_n || mm > A.max_m || nn < 0 || mm < 0) {
      flags |= ALN_RES_TOO_LONG;
    } else {
      n = (int)nn;
      m = (int)mm;
    }
    // the 16-bit kernel redoes these pairs in 32 bits (and no pair that it flags)
    bool redo = !FIXED && A.use16 && flags == 0 && MODE != ALN_LOCAL && !fits16(P, n, m, true);
    if (FIXED) {
      fw = A.fwd[p];
      flags |= fw.flags & (ALN_RES_BAD_CODE | ALN_RES_TOO_LONG | ALN_RES_DEVICE_ERROR);
      if (!flags && (fw.q_end < 0 || fw.q_end > n || fw.s_end < 0 || fw.s_end > m)) flags |= ALN_RES_BAD_END;
      n = flags ? 0 : fw.q_end;
      m = flags ? 0 : fw.s_end;
    }
    const uint8_t* __restrict__ q = A.q + qb;
    const uint8_t* __restrict__ s = A.s + sb;
    bool bad = false;
    int best = (MODE == ALN_GLOBAL && n + m > 0) ? P.go + (n + m) * P.ge : 0, bi = n, bj = m;
    if (n > 0 && m > 0) {
      int4 o = relax_pair<MODE, AFFINE, PROF, FA, FIXED>(P, tab, sig2, lds, q, n, s, m, lane, row, codes, bad);
      if constexpr (FIXED && PROF != kProfTable) {
        if (__any(bad))
          o = relax_pair<MODE, AFFINE, kProfTable, FA, FIXED>(P, tab, sig2, lds, q, n, s, m, lane, row, codes, bad);
      }
      best = o.x;
      if (!FIXED) {
        bi = o.y;
        bj = o.z;
        if (MODE == ALN_LOCAL && best <= 0) {
          best = bi = bj = 0;  // the empty alignment
        } else if (MODE == ALN_SEMIGLOBAL && best <= 0) {
          best = bi = 0;  // (0, m) precedes every other candidate in row-major order
          bj = m;
        }
      }
    } else {
      // an empty side: no cell is relaxed, so the other side's letters are checked here (its border is not a cell)
      for (int c = lane; c < n; c += 64) bad |= q[c] >= P.alphabet;
      for (int c = lane; c < m; c += 64) bad |= s[c] >= P.alphabet;
      if (!FIXED && MODE != ALN_GLOBAL) bi = bj = 0;
    }
    if (FIXED && !flags && best != fw.score) flags |= ALN_RES_BAD_END;
    if (__any(bad)) {
      flags |= ALN_RES_BAD_CODE;
      redo = false;
    }
    if (!FIXED && A.use16 && flags == 0 && MODE == ALN_LOCAL && best >= 32767) redo = true;
    aln_result_t res;
    res.score = flags ? 0 : best;
    res.q_begin = -1;
    res.q_end = flags ? 0 : bi;
    res.s_begin = -1;
    res.s_end = flags ? 0 : bj;
    res.cigar_len = 0;
    res.reserved = 0;
    if (!flags) {
      const int64_t c0 = A.cigar_off[p];
      const int64_t cap = A.cigar_off[p + 1] - c0;
      WalkState S;
      walk_start(S, bi, bj);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the codes are written before they are read
      walk_core<MODE>(codes, m, 0, 0, 0, S, reinterpret_cast<uint16_t*>(lds), lane, A.cigar + c0, cap);
      const int64_t runs = walk_finish(S, lane, A.cigar + c0, cap);
      res.q_begin = S.i;
      res.s_begin = S.j;
      res.cigar_len = (int)runs;
      if (runs > cap) flags |= ALN_RES_CIGAR_TRUNC;
      if (S.stuck) flags |= ALN_RES_DEVICE_ERROR;
    }
    res.flags = flags | (redo ? ALN_RES_INT32_REDO : 0u);
    if (lane == 0) A.out[p] = res;
    __builtin_amdgcn_wave_barrier();  // the wave stays together from pair to pair
  }
}

size_t row_bytes(int64_t m) { return ((size_t)(m + 1) * sizeof(int2) + 255) & ~(size_t)255; }
size_t code_bytes(int64_t n, int64_t m) {
  return ((size_t)((n + kWfR - 1) / kWfR) * (size_t)m * sizeof(uint16_t) + 255) & ~(size_t)255;
}

template <int MODE, bool AFFINE, int PROF, bool FA>
void launch_f(const KParams& kp, const WaveArgs& a, int waves, hipStream_t stream) {
  const int blocks = (waves + kPWavesPerBlock - 1) / kPWavesPerBlock;
  const size_t lds = (size_t)kPWavesPerBlock * pair_lds_bytes(kp.alphabet, PROF == kProfLane);
  const size_t rb = row_bytes(a.max_m), wb = rb + code_bytes(a.max_n, a.max_m);
  if (a.fwd)
    hipLaunchKernelGGL((batch_wave_kernel<MODE, AFFINE, PROF, FA, true>), dim3(blocks), dim3(64 * kPWavesPerBlock), lds,
                       stream, kp, a, waves, wb, rb);
  else
    hipLaunchKernelGGL((batch_wave_kernel<MODE, AFFINE, PROF, FA, false>), dim3(blocks), dim3(64 * kPWavesPerBlock), lds,
                       stream, kp, a, waves, wb, rb);
}

template <int MODE>
void launch_m(const KParams& kp, const WaveArgs& a, int waves, hipStream_t stream) {
  const bool bytes = score_bytes(kp);
  const bool fa = band_fits_fa(kp, a.max_n, a.max_m);
  auto go = [&](auto affine, auto lanes) {
    constexpr bool kAffine = decltype(affine)::value, kFa = decltype(lanes)::value;
    if (kAffine && !kFa)
      launch_f<MODE, kAffine, kProfTable, kFa>(kp, a, waves, stream);  // gap scores in the thousands
    else if (bytes && kp.alphabet <= 4)
      launch_f<MODE, kAffine, kAffine && !kFa ? kProfTable : kProfReg, kFa>(kp, a, waves, stream);
    else if (bytes)
      launch_f<MODE, kAffine, kAffine && !kFa ? kProfTable : kProfLane, kFa>(kp, a, waves, stream);
    else
      launch_f<MODE, kAffine, kProfTable, kFa>(kp, a, waves, stream);
  };
  if (kp.go == 0)
    go(std::false_type(), std::false_type());
  else if (fa)
    go(std::true_type(), std::true_type());
  else
    go(std::true_type(), std::false_type());
}

}  // namespace

// The rule compares both kernels' times, from what they measured (256 compute units).  One pair per wave: 0.128 ns for
// every step of every band and pair, 105 steps a band beyond its columns (65,536 reads of 100..250 letters 2.9 ms, of
// 20..30 letters 1.6 ms).  One pair per lane: a wave's largest pair alone, 56 ns a cell of it in 16 bits and 87 ns in 32, 1.65
// times that once two waves share a SIMD (reads of 100..250 letters 4.5 and 7.0 ms for up to 65,536 pairs, 8.1 ms for
// 262,144 in 16 bits); a batch that more than fills those waves stays with them.  Taken by the call's bounds, reads of
// 100..250 letters go one per wave up to 83,933 pairs (there 3.7 ms against 5.0 one per lane), of 8..30 up to 3111 (0.10 and 0.13).
// Local pairs, 20 letters and linear gaps gain more there (1.2 to 2.9 times), so the line could lie higher for them.
//
// The bounds may be far above the pairs' lengths, and then one wave per pair loses by as much as the lanes' largest pair is
// smaller than the bound (100,000 pairs of 8..30 letters under a bound of 1024: 1.47 ms one per wave, 0.20 per lane).  So above the
// number of pairs where every wave has one to itself, where it costs at most what the lanes do whatever the lengths
// (5000 pairs of 8..30 letters: 0.13 ms and 0.14), the pairs' own steps and largest cells are summed on the device and have to
// agree.  Both kernels are then launched, and the one that is not taken finds no pairs (20,011 reads of 100..250 letters traced back
// from their ends 720 us, 728 so; 60,000 with CIGARs 3.5 ms either way).
PairRoute wave_pair_route(int64_t n_pairs, int64_t lane_n, int64_t lane_m, size_t ws_bytes, bool use16) {
  PairRoute r{};
  const int cus = device_cu_count();
  if (cus <= 0 || n_pairs < 1 || lane_n < 1 || lane_m < 1) return r;
  const int64_t lane_waves = (n_pairs + (use16 ? 127 : 63)) / (use16 ? 128 : 64);
  if (use16 && lane_waves > (int64_t)8 * cus) return r;
  r.step_ns = 0.128 * 256 / cus;
  r.cell_ns = (use16 ? 56.0 : 87.0) *
              (lane_waves > (int64_t)4 * cus ? 1.65 * std::max(1.0, (double)lane_waves / (8 * cus)) : 1.0);
  if ((double)n_pairs * (double)wave_pair_steps(lane_n, lane_m) * r.step_ns > (double)lane_pair_cells(lane_n, lane_m) * r.cell_ns)
    return r;
  const int64_t all = (int64_t)cus * kPWavesPerCU;
  r.measure = n_pairs > all;
  const int64_t fit = (int64_t)(ws_bytes / (row_bytes(lane_m) + code_bytes(lane_n, lane_m)));
  r.waves = (int)std::min(std::min(n_pairs, all), fit);
  return r;
}

// The work of one part of aln_traceback's pairs: the rectangles up to their end cells.
__global__ __launch_bounds__(256) void pair_work_kernel(const WaveArgs A, PairWork* __restrict__ work) {
  __shared__ PairWork s_work;
  if (threadIdx.x == 0) s_work.steps = s_work.cells = 0;
  __syncthreads();
  unsigned long long steps = 0, cells = 0;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < A.n_pairs; p += (int64_t)gridDim.x * blockDim.x) {
    // (an end cell outside the pair is flagged by the kernels, and within the bounds it does no harm here)
    const int n = A.fwd[p].q_end, m = A.fwd[p].s_end;
    if (n < 0 || m < 0 || n > A.max_n || m > A.max_m) continue;
    steps += (unsigned long long)wave_pair_steps(n, m);
    cells = max(cells, (unsigned long long)lane_pair_cells(n, m));
  }
  const PairWork w = wave_work({steps, cells});
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&s_work.steps, w.steps);
    atomicMax(&s_work.cells, w.cells);
  }
  __syncthreads();
  if (threadIdx.x == 0) work[blockIdx.x] = s_work;
}

void launch_pair_work(const WaveArgs& a, PairWork* work, hipStream_t stream) {
  hipLaunchKernelGGL(pair_work_kernel, dim3(kWorkSlots), dim3(256), 0, stream, a, work);
}

aln_status_t launch_batch_wave(const KParams& kp, const WaveArgs& a, int waves, hipStream_t stream) {
  ProfScope prof(a.fwd ? "batch_wave_traceback_from_end" : "batch_wave_traceback", stream);
  switch (kp.mode) {
    case ALN_GLOBAL:
      launch_m<ALN_GLOBAL>(kp, a, waves, stream);
      break;
    case ALN_LOCAL:
      launch_m<ALN_LOCAL>(kp, a, waves, stream);
      break;
    default:
      launch_m<ALN_SEMIGLOBAL>(kp, a, waves, stream);
      break;
  }
  return hipGetLastError() == hipSuccess ? ALN_OK : ALN_E_DEVICE;
}

}  // namespace mialign
