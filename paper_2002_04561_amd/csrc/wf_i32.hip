// Intra-sequence wavefront engine, 32-bit lanes: bands of rows relaxed as anti-diagonal fronts.
//
// A work item is one band (BH = 64*R rows) of one pair.  A wave relaxes a band: lane l owns R
// consecutive rows and works on column j = t - l + 1 at step t, so the 64 lanes sweep the band as an
// anti-diagonal front (cells on one anti-diagonal are independent, AnySeq Sec. III-A).  The lane
// above hands its bottom-row H and E down with a DPP wave_shr:1 move each step; lane 0 takes the band's
// top row from LDS, every lane reads its column letters from an LDS window, and lane 63 writes its bottom
// row to LDS 4 columns at a time (a DPP shift register took two moves a step, a DPP chain for the letters one).
//
// Work is handed out in groups of kWfWavesPerBlock consecutive items from one atomic ticket, so
// several pairs of different sizes share the device the way the paper's dynamic wavefront shares
// its queue between alignments (Sec. IV-A).  A workgroup relaxes one group: its compute waves take
// the group's bands, and the band below of a pair reads the band above's bottom row from an LDS ring
// with LDS progress counters -- the tile border publication of Sec. IV-B, without device memory.
// Where a pair continues into the next group, the workgroup's courier wave copies the last band's
// row to the pair's row slot in HBM and publishes a per-band progress counter once the stores have
// completed (device-coherent sc1 accesses); the next group's courier streams it into its first
// band's ring.  Only couriers wait on device memory, so the compute waves run at the rate of the
// recurrence.  Groups are handed out in order, so every group a courier waits on is already running;
// every wait is bounded -- a wave that waits too long raises an error flag and leaves its band, and
// all waves still meet at the group's barriers, so the grid always drains.
#include <type_traits>

#include "internal.h"
#include "band.h"
#include "band_wave.h"
#include "walk.h"
#include "walk_wave.h"

namespace mialign {
namespace {

// A workgroup is a group of kWfWavesPerBlock compute waves, which relax consecutive bands, plus one
// courier wave.  Consecutive bands of a pair hand their rows to each other through LDS rings; the
// courier streams the group's first input row from HBM and its last output row to HBM, so only the
// courier ever waits on device memory.
constexpr int kWfWavesPerBlock = kWfGroupBands;       // compute waves (bands) per workgroup
constexpr int kWfBlock = 64 * (kWfWavesPerBlock + 1);  // plus the courier
constexpr int kRing = 256;                            // columns held by one LDS ring
constexpr int kBlkGrouped = 32;                       // steps between lane-0 input refills, grouped
constexpr int kCourierChunk = 32;                     // columns a courier moves between HBM and LDS at once
constexpr int kWfBlockAlone = 64 * kWfWavesPerBlock;  // bands on their own: no courier


__device__ __forceinline__ int dpp_shr1(int old, int src) {
  return __builtin_amdgcn_update_dpp(old, src, 0x138, 0xf, 0xf, false);  // wave_shr:1, lane 0 keeps old
}
__device__ __forceinline__ int dpp_shl1(int old, int src) {
  return __builtin_amdgcn_update_dpp(old, src, 0x130, 0xf, 0xf, false);  // wave_shl:1, lane 63 keeps old
}

// Packed 16-bit bands (local alignment, score only; register profiles for up to 4 letters, per-lane LDS
// profiles of two 16-bit rows per half for up to 32).  A 32-bit lane
// register holds two 16-bit cells: rows of the band's upper half (HB = 128 rows) in its low half and
// rows of the lower half in its high half, the lower half running kP16Delay steps behind so that the
// two are independent within a step -- the two halves are independent submatrices sharing one vector
// lane, as in the paper's inter-task vectorisation (Sec. IV-A), and each keeps its scores as 16-bit
// differences from an offset of its own, as the paper does within a block (Sec. IV-A): the offset is
// the half's top-row score at the first column of each block of steps.
typedef short s2 __attribute__((ext_vector_type(2)));
constexpr int kP16Half = 128;   // rows per half band
constexpr int kP16Delay = 96;   // steps between the upper and the lower half
constexpr int kDelayRing = 256; // columns of the upper half's bottom row kept for the lower half
constexpr int kNeg16 = -32768;  // stands for -infinity; sums saturate, so it stays far below real scores
// The lower half's lane 0 reads columns up to j + kBlkGrouped - 1 - kP16Delay at the start of the block
// of step j; the upper half's lane 63 has written them by then only if the delay covers a block plus
// lane 63's 63 steps.  The delay line must also keep a column until the lower half has read it.
static_assert(kP16Delay >= kBlkGrouped + 63, "the delay between the halves must cover a block and the lanes");
static_assert(kDelayRing >= kP16Delay + kBlkGrouped, "the delay line must hold the columns in flight");

__device__ __forceinline__ s2 as_s2(int x) { return __builtin_bit_cast(s2, x); }
__device__ __forceinline__ int as_int(s2 x) { return __builtin_bit_cast(int, x); }
__device__ __forceinline__ int sat16(int x) { return min(max(x, -32768), 32767); }
__device__ __forceinline__ int pack16(int lo, int hi) { return (int)(((uint32_t)lo & 0xffffu) | ((uint32_t)hi << 16)); }
__device__ __forceinline__ int lo16(int x) { return (int)(int16_t)(x & 0xffff); }
__device__ __forceinline__ int hi16(int x) { return x >> 16; }
__device__ __forceinline__ int padd(int a, int b) { return as_int(__builtin_elementwise_add_sat(as_s2(a), as_s2(b))); }
__device__ __forceinline__ int psub(int a, int b) { return as_int(__builtin_elementwise_sub_sat(as_s2(a), as_s2(b))); }
__device__ __forceinline__ int pmax(int a, int b) { return as_int(__builtin_elementwise_max(as_s2(a), as_s2(b))); }
// a 16-bit relative score back to an absolute 32-bit one (-infinity stays -infinity)
__device__ __forceinline__ int unrel16(int rel, int base) { return rel == kNeg16 ? kNeg32 : rel + base; }

// Bands on their own (one wave per band, hand-offs through HBM), handed out level by level (wf_order_kernel).
// The recurrence is band.h's.  A wave's stage holds its top-row inputs of 64 steps, H~ and E~ of column j at
// (j - 1) & 63; lane 63 writes its bottom row into the slots just consumed, a column late so that 4 columns are
// one aligned store: after the block's step t the slots hold columns up to t - 62.
template <int MODE, bool AFFINE, int PROF, bool TB, bool FA, int R>
__global__ __launch_bounds__(kWfBlockAlone, 4) void wf_i32_kernel(const KParams P, const uint8_t* __restrict__ Q,
                                                          const uint8_t* __restrict__ S, WfWs W) {
  static_assert(!lane_words(PROF) || R == 4, "a lane profile word holds 4 rows");
  __shared__ int32_t tab[PROF == kProfTable ? kTab * kTab : 1];
  __shared__ int4 stage[kWfWavesPerBlock][2][16];
  __shared__ LetterWindow<64> letters[kWfWavesPerBlock];
  extern __shared__ uint32_t lprof[];  // lane words: [wave][letter][lane], alphabet letters and the pad letter
  __shared__ uint32_t sig2[PROF == kProfTable ? 1 : kScoreWords];
  fill_table<PROF>(P, tab, sig2);
  __syncthreads();
  constexpr int BH = 64 * R;
  const int lane = threadIdx.x & 63;
  const int wib = threadIdx.x >> 6;
  int* st_h = reinterpret_cast<int*>(&stage[wib][0][0]);
  int* st_e = reinterpret_cast<int*>(&stage[wib][1][0]);
  LetterWindow<64>& lett = letters[wib];
  uint32_t* __restrict__ lp = lprof + (lane_words(PROF) ? wib * (P.alphabet + 1) * 64 + lane : 0);
  const int np = *W.n_pairs;
  const int64_t n_items = *W.n_items;

  // A batch whose pairs all have one band needs no ticket: no band waits on another and they come largest first, so
  // the waves take them in turn.  One ticket counter serves an atomic every 38 ns or so: 100,003 one-band pairs took
  // 3.9 ms whatever the bands cost.
  const bool in_turn = W.lv[0] <= 1;
  int64_t turn = (int64_t)blockIdx.x * kWfWavesPerBlock + wib;
  for (;;) {
    // The whole wave comes back here before lane 0 takes the next ticket.  Without a convergent operation in this
    // block the compiler may join lane 0's store at the end of a band with its atomic below and send the other
    // lanes straight to the shuffle, which then reads an inactive lane: they relax item 0 for ever.
    __builtin_amdgcn_wave_barrier();
    int64_t t = turn;
    if (!in_turn) {
      t = 0;
      if (lane == 0) t = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(W.ticket), 1ull);
      t = __shfl(t, 0, 64);
    }
    turn += (int64_t)gridDim.x * kWfWavesPerBlock;
    if (t >= n_items) break;
    if (__hip_atomic_load(W.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
    t = W.order[t];  // the item (pair-major band index) this ticket hands out
    const WfPair pr = W.pairs[np == 1 ? 0 : W.item_pair[t]];
    const int b = __builtin_amdgcn_readfirstlane((int)(t - pr.item0));
    const int n = __builtin_amdgcn_readfirstlane(pr.n), m = __builtin_amdgcn_readfirstlane(pr.m);
    const int nb = __builtin_amdgcn_readfirstlane(pr.nb);
    // rows come from the query array, columns from the subject array, or the reverse when flipped
    const bool flip = __builtin_amdgcn_readfirstlane(pr.flip) != 0;
    const uint8_t* __restrict__ q = (flip ? S : Q) + pr.q_off;
    const uint8_t* __restrict__ s = (flip ? Q : S) + pr.s_off;
    const int64_t ld = (int64_t)m + 1;

    const int i0 = b * BH, irow0 = i0 + lane * R;
    int prof[R];
    BandLane<R> L;
    BandBest<R> B;
    bool bad = false;
    band_start<MODE, PROF, FA, R>(P, sig2, q, n, flip, irow0, lane, lp, prof, L, B, bad);
    uint16_t* __restrict__ codes = TB ? W.codes + pr.code_off + (size_t)(b * 64 + lane) * (size_t)m : nullptr;
    const bool last_band = (b == nb - 1);
    if (MODE == ALN_SEMIGLOBAL && last_band) last_row_start<R>(P, n - 1 - irow0, B);
    int2* __restrict__ prev = W.rows + pr.row_off + (int64_t)((b + 1) & 1) * ld;
    int2* __restrict__ cur = W.rows + pr.row_off + (int64_t)(b & 1) * ld;
    bool failed = false;

    int seen = 0;  // columns of the previous band known to be published
    constexpr int BLK = 64;
    // letters are loaded one block ahead; those of columns before the first are pad letters
    int c_next = 1 + lane <= m ? (int)s[lane] : -1;
    int c_idx = letter_index<PROF, R>(P, -1, flip, bad);
    lett.clear_tail(lane);

    const int steps = m + 64;  // lane 63's column m leaves at step m + 63
    for (int tb = 0; tb < steps; tb += BLK) {
      // lane-0 inputs for steps tb..tb+63 (columns tb+1..tb+64)
      const int col_in = tb + 1 + lane;
      const int c_old = c_idx;
      c_idx = letter_index<PROF, R>(P, c_next, flip, bad);
      lett.put(lane, c_old, c_idx);
      c_next = col_in + BLK <= m ? (int)s[col_in + BLK - 1] : -1;
      int32_t th = lane_neg<FA>(), te = lane_neg<FA>();
      if (b == 0) {
        if (col_in <= m) th = border_h<MODE, FA>(P, 0, col_in);
      } else {
        const int need = min(tb + BLK, m);
        if (seen < need) {
          int v = 0;
          if (lane == 0) {
            long long spins = 0;
            for (;;) {
              v = __hip_atomic_load(W.flags + (t - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              if (v >= need) break;
              if (++spins > P.spin_dev || __hip_atomic_load(W.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                v = -1;
                break;
              }
              __builtin_amdgcn_s_sleep(1);
            }
          }
          v = __shfl(v, 0, 64);
          if (v < 0) {
            if (lane == 0) __hip_atomic_store(W.error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            failed = true;
            break;
          }
          // The row data below is read with device-coherent (sc1) loads issued after the flag load has
          // returned, so they observe the producer's sc1 stores that completed before its flag store.
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          seen = v;
        }
        if (col_in <= m) {
          const long long pv = __hip_atomic_load(reinterpret_cast<long long*>(prev + col_in), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
          th = (int32_t)(pv & 0xffffffffll);
          te = (int32_t)(pv >> 32);
        }
      }
      if (MODE == ALN_LOCAL)
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
          band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupInside>(P, tab, prof, I, j0, m, L, G, [](int) {});
        else
          band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupStart>(P, tab, prof, I, j0, m, L, G, [](int) {});
        if (MODE != ALN_LOCAL && t0 + 4 >= m)
          track_last_column<FA, R, MODE == ALN_GLOBAL>(P, G, j0, n, m, irow0, B);
        if (TB) store_codes<R>(G, codes, j0, m, inside);
        if constexpr (MODE == ALN_LOCAL) track_local<AFFINE, R>(P, L, G, floor0, j0, flip, B);
        if (MODE == ALN_SEMIGLOBAL && last_band) track_last_row<AFFINE, R>(P, L, G, floor0, m, n - 1 - i0, j0, B);
        if (lane == 63) {
          reinterpret_cast<int4*>(st_h)[g4] = make_int4(ph, G.oh[0], G.oh[1], G.oh[2]);
          reinterpret_cast<int4*>(st_e)[g4] = make_int4(pe, G.oe[0], G.oe[1], G.oe[2]);
        }
      };
      run_block<PROF, R, BLK / 4>(lett, lp, lane, min(BLK / 4, (steps - tb + 3) / 4), load_rows, run);
      // slot u now holds lane 63's column tb + u - 63
      if (b + 1 < nb) {
        const int col_out = tb + lane - 63;
        if (col_out >= 1 && col_out <= m) {
          const long long pv = ((long long)(uint32_t)st_h[lane]) | ((long long)st_e[lane] << 32);
          __hip_atomic_store(reinterpret_cast<long long*>(cur + col_out), pv, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        }
        const int published = min(tb, m);
        // Publication: the row stores above are device-coherent (sc1) atomics; waiting for their
        // completion before the sc1 flag store orders them without an L2 write-back (an agent-scope
        // release fence would emit buffer_wbl2 on every publication).
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (published >= 1 && lane == 0)
          __hip_atomic_store(W.flags + t, published, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    const int4 opt = band_optimum<MODE, FA, R>(P, B, n, m, flip, last_band, irow0, bad, failed);
    if (lane == 0) W.band_res[t] = opt;
  }
}

// Bands in groups (workgroups of kWfWavesPerBlock bands and a courier), same recurrence.  A ring holds H~ and E~
// of column j at (j - 1) mod kRing; a band reads its top row straight from its ring, 4 columns at a time, and lane
// 63 writes the bottom row into the next ring as it goes, a column late so that 4 columns are one aligned store.
// CKPT: also store checkpoints for a linear-space traceback (one pair, groups aligned with its bands):
// every group's bottom row stays in its own row slot instead of two rotating ones, and every
// kTileCols-th column's H~ and F~ of all rows go to W.ckcols.
// WAVES: the waves a SIMD it is built for.  5 leave 96 registers, so a group's inputs are read when it starts and not a group
// ahead: for launches of more workgroups than are resident at 4 (SplitPlan::crowded).  Short chains of bands wait
// along the chain for most of their time, and then the number of chains in flight is what counts: 4096 pairs of 1024 x 64 letters,
// global affine 0.50 and 0.43 ms, semi-global linear 0.55 and 0.44, 4096 of 512 x 1600 (local) 0.98 and 0.87.  With a workgroup or
// two a compute unit 4 is better: 1024 pairs of 512 x 1600 0.32 and 0.40.
template <int MODE, bool AFFINE, int PROF, bool TB, bool FA, int R, bool P16, bool CKPT, int WAVES>
__global__ __launch_bounds__(kWfBlock, WAVES) void wf_i32_group_kernel(const KParams P, const uint8_t* __restrict__ Q,
                                                          const uint8_t* __restrict__ S, WfWs W) {
  static_assert(!lane_words(PROF) || R == 4, "a lane profile word holds 4 rows");
  constexpr int BLK = kBlkGrouped;
  // packed bands: sigma - ge by (query letter, subject letter), the source of their profiles; kProfTable: sigma - 2 ge
  __shared__ int32_t tab[P16 || PROF == kProfTable ? kTab * kTab : 1];
  __shared__ uint32_t sig2[P16 || PROF == kProfTable ? 1 : kScoreWords];
  __shared__ int4 stage[P16 ? kWfWavesPerBlock : 1][3][BLK / 4];  // packed bands: lane-0 inputs of BLK steps
  __shared__ LetterWindow<BLK> letters[P16 ? 1 : kWfWavesPerBlock];
  // ring k carries the rows feeding compute wave k; ring kWfWavesPerBlock feeds the courier
  __shared__ int4 ring4[kWfWavesPerBlock + 1][2][kRing / 4];
  __shared__ int pub[kWfWavesPerBlock + 1];  // columns written into each ring
  __shared__ int con[kWfWavesPerBlock + 1];  // columns read out of each ring
  __shared__ long long s_t0;                 // first item of the group
  __shared__ int s_err;
  extern __shared__ uint32_t lprof[];        // lane words: [wave][letter][lane], alphabet letters and the pad letter
  static_assert(!P16 || (MODE == ALN_LOCAL && (PROF == kProfReg || PROF == kProfLane) && !TB && R == 4),
                "packed bands: local, score only, register or per-lane profiles");
  static_assert(!CKPT || (!TB && !P16 && R == 4), "checkpoints: 32-bit score-only bands");
  // packed bands: the upper half's bottom row (absolute H, E) on its way to the lower half
  __shared__ int2 dline[P16 ? kWfWavesPerBlock : 1][P16 ? kDelayRing : 1];
  if constexpr (P16) {
    for (int k = threadIdx.x; k < kTab * kTab; k += blockDim.x) {
      const int a = k / kTab, b = k % kTab;
      tab[k] = (a >= P.alphabet || b >= P.alphabet) ? -kBig32 : (int32_t)P.sig[a * kMaxAlphabet + b] - P.ge;
    }
  } else {
    fill_table<PROF>(P, tab, sig2);
  }
  __syncthreads();
  constexpr int BH = 64 * R;
  const int lane = threadIdx.x & 63;
  const int wib = threadIdx.x >> 6;
  const int cw = wib < kWfWavesPerBlock ? wib : 0;  // the courier borrows wave 0's pointers
  [[maybe_unused]] const int32_t go = P.go, ge = P.ge, goe = P.goe;
  const int np = *W.n_pairs;
  const int64_t n_items = *W.n_items;
  auto ring_h = [&](int k) -> int* { return reinterpret_cast<int*>(&ring4[k][0][0]); };
  auto ring_e = [&](int k) -> int* { return reinterpret_cast<int*>(&ring4[k][1][0]); };

  // Bounded waits.  A wave that gives up raises the group's and the launch's error flags and leaves
  // its band; every wave still meets the group's barriers, so the grid drains.
  auto give_up = [&]() {
    if (lane == 0) {
      __hip_atomic_store(&s_err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_store(W.error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto lds_wait_ge = [&](int* p, int v) -> bool {
    long long spins = 0;
    while (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < v) {
      __builtin_amdgcn_s_sleep(1);
      if (++spins > P.spin_lds || __hip_atomic_load(&s_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
        give_up();
        return false;
      }
    }
    return true;
  };

  // The courier: for the group's first band (if it has a band above, in another group) it streams
  // that band's bottom row from HBM into ring 0, kCourierChunk columns at a time, once the band above has
  // published them; for the group's last band (if its band below is in another group) it copies
  // ring kWfWavesPerBlock to the pair's row slot in HBM and publishes the band's progress counter
  // once those stores have completed.  HBM rows and counters use device-coherent (sc1) accesses.
  auto courier = [&](int64_t t0) {
    const int64_t tin = t0, tout = t0 + kWfWavesPerBlock - 1;
    bool in_on = false, out_on = false;
    int m_in = 0, m_out = 0;
    const int2* src = nullptr;
    int2* dst = nullptr;
    if (tin < n_items) {
      const WfPair a = W.pairs[np == 1 ? 0 : W.item_pair[tin]];
      const int b = (int)(tin - a.item0);
      if (b > 0) {
        in_on = true;
        m_in = a.m;
        const int64_t slot = CKPT ? b / kWfWavesPerBlock - 1 : ((b + 1) & 1);
        src = W.rows + a.row_off + slot * ((int64_t)a.m + 1);
      }
    }
    if (tout < n_items) {
      const WfPair a = W.pairs[np == 1 ? 0 : W.item_pair[tout]];
      const int b = (int)(tout - a.item0);
      if (b + 1 < a.nb) {
        out_on = true;
        m_out = a.m;
        const int64_t slot = CKPT ? b / kWfWavesPerBlock : (b & 1);
        dst = W.rows + a.row_off + slot * ((int64_t)a.m + 1);
      }
    }
    int in_done = 0, out_done = 0, seen = 0;
    long long idle = 0;
    while ((in_on && in_done < m_in) || (out_on && out_done < m_out)) {
      bool moved = false;
      if (in_on && in_done < m_in) {
        const int want = min(in_done + kCourierChunk, m_in);
        if (seen < want) seen = __hip_atomic_load(W.flags + (tin - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (seen >= want &&
            __hip_atomic_load(&con[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= want - kRing) {
          // the row loads are issued after the counter load has returned (device-coherent loads)
          const int col = in_done + 1 + lane;
          if (col <= want) {
            const long long v = __hip_atomic_load(reinterpret_cast<const long long*>(src + col), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
            ring_h(0)[(col - 1) % kRing] = (int32_t)(v & 0xffffffffll);
            ring_e(0)[(col - 1) % kRing] = (int32_t)(v >> 32);
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (lane == 0) __hip_atomic_store(&pub[0], want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          in_done = want;
          moved = true;
        }
      }
      if (out_on && out_done < m_out) {
        const int want = min(out_done + kCourierChunk, m_out);
        if (__hip_atomic_load(&pub[kWfWavesPerBlock], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= want) {
          const int col = out_done + 1 + lane;
          if (col <= want) {
            const int vh = ring_h(kWfWavesPerBlock)[(col - 1) % kRing], ve = ring_e(kWfWavesPerBlock)[(col - 1) % kRing];
            const long long pv = ((long long)(uint32_t)vh) | ((long long)ve << 32);
            __hip_atomic_store(reinterpret_cast<long long*>(dst + col), pv, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          }
          // stores complete (device-coherent) before the counter that announces them; the ring
          // values were read before the stores were issued, so the slots can be released too
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          if (lane == 0) {
            __hip_atomic_store(W.flags + tout, want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&con[kWfWavesPerBlock], want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          out_done = want;
          moved = true;
        }
      }
      if (moved) {
        idle = 0;
      } else {
        __builtin_amdgcn_s_sleep(1);
        if (++idle > P.spin_dev || __hip_atomic_load(&s_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ||
            __hip_atomic_load(W.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          give_up();
          break;
        }
      }
    }
  };


  // Packed 16-bit band t (see kP16Half): lane l holds rows i0 + 2l + 1, i0 + 2l + 2 of the upper half
  // in the low 16 bits and the same rows plus kP16Half in the high 16 bits.  The upper half works on
  // column j = t - l + 1 at step t, the lower half on j - kP16Delay.  Values are the row-biased Hb of
  // the 32-bit kernel minus the half's offset; each block re-bases both halves on their top-row
  // scores at the block's first column, so every value of a block stays within a few thousand of its
  // offset (adjacent cells differ by at most max|sigma| + |go| + 2|ge|, which the host bounds).  The
  // band's inputs and outputs are absolute 32-bit rows, as for the 32-bit bands.
  [[maybe_unused]] auto p16_band = [&](auto t_) {
    const int64_t t = t_;
    int* st_h = reinterpret_cast<int*>(&stage[cw][0][0]);
    int* st_e = reinterpret_cast<int*>(&stage[cw][1][0]);
    int* st_c = reinterpret_cast<int*>(&stage[cw][2][0]);
    const WfPair pr = W.pairs[np == 1 ? 0 : W.item_pair[t]];
    const int b = (int)(t - pr.item0);
    const int n = pr.n, m = pr.m, nb = pr.nb;
    const bool flip = pr.flip != 0;
    const uint8_t* __restrict__ q = (flip ? S : Q) + pr.q_off;
    const uint8_t* __restrict__ s = (flip ? Q : S) + pr.s_off;
    auto sig_rc = [&](int cr, int cc) -> int { return flip ? tab[cc * kTab + cr] : tab[cr * kTab + cc]; };
    constexpr int HB = kP16Half, D = kP16Delay, BH = 64 * R;
    const int i0 = b * BH;
    // half h (0 upper, 1 lower), row r (0, 1): i = i0 + h * HB + 2 lane + r + 1
    int prof[2][2];
    int rowc[2][2];
    int32_t nuA[2][2], bvA[2][2];
    int bjA[2][2];
    bool bad = false;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int i = i0 + h * HB + 2 * lane + r + 1;
        int c = kPad;
        if (i <= n) {
          c = q[i - 1];
          if (c >= P.alphabet) {
            bad = true;
            c = kPad;
          }
        }
        rowc[h][r] = c;
        uint32_t w = 0;
        if (PROF == kProfReg) {
          for (int a = 0; a < 4; ++a) {
            const int v = (c < P.alphabet && a < P.alphabet) ? sig_rc(c, a) : -128;
            w |= ((uint32_t)(v & 0xff)) << (8 * a);
          }
        }
        prof[h][r] = (int)w;
        nuA[h][r] = -i * ge;  // Hb(i, j) of H = 0, also Hb(i, 0)
        bvA[h][r] = kNeg32;
        bjA[h][r] = 0;
      }
    // kProfLane: per column letter, this lane's two rows of each half as 16-bit sigma - ge, the upper
    // half's in lpu[letter * 64] and the lower half's in lpl[letter * 64]; each lane reads only its own
    // words, so no barrier
    const uint32_t* __restrict__ lpu = lprof + (PROF == kProfLane ? (size_t)wib * 2 * P.alphabet * 64 + lane : 0);
    const uint32_t* __restrict__ lpl = lpu + (PROF == kProfLane ? (size_t)P.alphabet * 64 : 0);
    if (PROF == kProfLane) {
      uint32_t* wu = lprof + (size_t)wib * 2 * P.alphabet * 64 + lane;
      for (int a = 0; a < P.alphabet; ++a) {
        uint32_t hw[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int v0 = rowc[h][0] < P.alphabet ? sig_rc(rowc[h][0], a) : -128;
          const int v1 = rowc[h][1] < P.alphabet ? sig_rc(rowc[h][1], a) : -128;
          hw[h] = (uint32_t)(v0 & 0xffff) | ((uint32_t)v1 << 16);
        }
        wu[a * 64] = hw[0];
        wu[(P.alphabet + a) * 64] = hw[1];
      }
    }
    int32_t B0 = -i0 * ge, B1 = -(i0 + HB) * ge;  // offsets: Hb of each half's top row at column 0
    int hl[2], f[2], nu[2], bvr[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      hl[r] = pack16(sat16(nuA[0][r] - B0), sat16(nuA[1][r] - B1));
      f[r] = pack16(kNeg16, kNeg16);
      nu[r] = hl[r];
      bvr[r] = pack16(kNeg16, kNeg16);
    }
    int diag = pack16(sat16(-(i0 + 2 * lane) * ge - B0), sat16(-(i0 + HB + 2 * lane) * ge - B1));
    int bot_h = 0, bot_e = pack16(kNeg16, kNeg16), cur_c = 0, out_h = 0, out_e = 0;
    const int go2 = pack16(go, go), ge2 = pack16(ge, ge), goe2 = pack16(goe, goe);
    bool failed = false;
    int *rin_h = ring_h(wib), *rin_e = ring_e(wib), *rout_h = ring_h(wib + 1), *rout_e = ring_e(wib + 1);
    int2* __restrict__ dl = dline[wib];
    const bool has_out = b + 1 < nb;
    auto letter_raw = [&](int col) -> int { return (col >= 1 && col <= m) ? (int)s[col - 1] : -1; };
    auto letter_idx = [&](int c) -> int {
      if (c < 0) return 0;
      if (c >= P.alphabet) {
        bad = true;
        c = 0;
      }
      return PROF == kProfLane ? c * 64 : c * 8;
    };
    int cn0 = lane < BLK ? letter_raw(1 + lane) : -1;
    int cn1 = lane < BLK ? letter_raw(1 + lane - D) : -1;

    const int steps = m + 63 + D;  // lane 63's lower half reaches column m at step m + 62 + D
    for (int tb = 0; tb < steps; tb += BLK) {
      const int col0 = tb + 1 + lane, col1 = col0 - D;  // lane-0 input columns of the two halves
      const int c0 = letter_idx(cn0), c1 = letter_idx(cn1);
      asm volatile("" ::"v"(c0), "v"(c1) : "memory");
      cn0 = lane < BLK ? letter_raw(col0 + BLK) : -1;
      cn1 = lane < BLK ? letter_raw(col1 + BLK) : -1;
      int32_t th0 = 0, te0 = kNeg32, th1 = 0, te1 = kNeg32;
      if (b > 0) {
        const int need = min(tb + BLK, m);
        if (!lds_wait_ge(&pub[wib], need)) {
          failed = true;
          break;
        }
        if (lane < BLK && col0 <= m) {
          th0 = rin_h[(col0 - 1) % kRing];
          te0 = rin_e[(col0 - 1) % kRing];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_store(&con[wib], need, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      if (lane < BLK && col1 >= 1 && col1 <= m) {
        const int2 v = dl[col1 % kDelayRing];
        th1 = v.x;
        te1 = v.y;
      }
      // re-base each half on its top-row score at the block's first column while it is in the matrix
      const int nB0 = (tb + 1 <= m) ? __builtin_amdgcn_readfirstlane(th0) : B0;
      const int nB1 = (tb + 1 - D >= 1 && tb + 1 - D <= m) ? __builtin_amdgcn_readfirstlane(th1) : B1;
      if (nB0 != B0 || nB1 != B1) {
        const int dd = pack16(sat16(nB0 - B0), sat16(nB1 - B1));
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          hl[r] = psub(hl[r], dd);
          f[r] = psub(f[r], dd);
        }
        bot_h = psub(bot_h, dd);
        bot_e = psub(bot_e, dd);
        diag = psub(diag, dd);
        B0 = nB0;
        B1 = nB1;
      }
      {
        // floors (see raise_local_floor): the best of both halves' top-row inputs and recorded optima
        int v = max(th0 + i0 * ge, th1 + (i0 + HB) * ge);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 2; ++r) v = max(v, bvA[h][r] - nuA[h][r]);
        const int fl = __ockl_wfred_max_i32(v) - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 2; ++r) bvA[h][r] = max(bvA[h][r], fl + nuA[h][r]);
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        nu[r] = pack16(sat16(nuA[0][r] - B0), sat16(nuA[1][r] - B1));
        bvr[r] = pack16(sat16(bvA[0][r] - B0), sat16(bvA[1][r] - B1));
      }
      if (lane < BLK) {
        st_h[lane] = pack16(sat16(th0 - B0), sat16(th1 - B1));
        st_e[lane] = pack16(sat16(te0 - B0), sat16(te1 - B1));
        st_c[lane] = c0 | (c1 << 16);
      }
      // One step: lane l relaxes its two rows of each half, the upper at column j = tt - l + 1 and the
      // lower at j - D.  Near the matrix edges (CK) a half outside it keeps its state unchanged.
      auto step = [&](int tt, int in_top_h, int in_top_e, int in_top_c, auto checked, int* hk) {
        constexpr bool CK = decltype(checked)::value;
        const int j0 = tt - lane + 1, j1 = j0 - D;
        const int in_h = dpp_shr1(in_top_h, bot_h);
        const int in_e = dpp_shr1(in_top_e, bot_e);
        const int in_c = dpp_shr1(in_top_c, cur_c);
        cur_c = in_c;
        const int c1s = (int)((uint32_t)in_c >> 16);
        const uint32_t wu = PROF == kProfLane ? lpu[in_c & 0xffff] : 0u;
        const uint32_t wl = PROF == kProfLane ? lpl[c1s] : 0u;
        const bool ok0 = !CK || (j0 >= 1 && j0 <= m), ok1 = !CK || (j1 >= 1 && j1 <= m);
        const int keep = (ok0 ? 0 : 0xffff) | (ok1 ? 0 : (int)0xffff0000u);  // bits left unchanged
        auto sel = [&](int old, int nw) { return CK ? ((keep & old) | (~keep & nw)) : nw; };
        int hd = diag, hup = in_h, eup = in_e;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const int hlo = hl[r];
          const int e = AFFINE ? pmax(eup, padd(hup, go2)) : hup;
          const int ff = AFFINE ? pmax(padd(f[r], ge2), padd(hlo, goe2)) : padd(hlo, ge2);
          // sigma - ge of both halves' cells side by side: register bytes picked by bit-field extracts
          // (kProfReg), or the 16-bit halves of the two halves' profile words (kProfLane)
          int sg;
          if constexpr (PROF == kProfLane) {
            sg = (int)__builtin_amdgcn_perm(wl, wu, r ? 0x07060302u : 0x05040100u);
          } else {
            sg = (int)__builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_sbfe(prof[1][r], c1s, 8),
                                            (uint32_t)__builtin_amdgcn_sbfe(prof[0][r], in_c, 8), 0x05040100u);
          }
          const int d = padd(hd, sg);
          const int h = pmax(pmax(d, pmax(e, ff)), nu[r]);
          if (CK) {
            // exact cell-by-cell optimum tracking, per half
            const int v0 = lo16(h), v1 = hi16(h);
            if (ok0 && v0 > lo16(bvr[r])) {
              bvA[0][r] = v0 + B0;
              bjA[0][r] = j0;
              bvr[r] = pack16(v0, hi16(bvr[r]));
            }
            if (ok1 && v1 > hi16(bvr[r])) {
              bvA[1][r] = v1 + B1;
              bjA[1][r] = j1;
              bvr[r] = pack16(lo16(bvr[r]), v1);
            }
          } else {
            hk[r] = h;
          }
          f[r] = sel(f[r], ff);
          hl[r] = sel(hlo, h);
          hd = hlo;
          hup = h;
          eup = e;
        }
        bot_h = sel(bot_h, hup);
        bot_e = sel(bot_e, eup);
        diag = sel(diag, in_h);
        out_h = dpp_shl1(bot_h, out_h);
        out_e = dpp_shl1(bot_e, out_e);
      };
      for (int g4 = 0; g4 < BLK / 4; ++g4) {
        const int t0 = tb + 4 * g4;
        const int4 vh = reinterpret_cast<const int4*>(st_h)[g4];
        const int4 ve = reinterpret_cast<const int4*>(st_e)[g4];
        const int4 vc = reinterpret_cast<const int4*>(st_c)[g4];
        if (t0 >= 63 + D && t0 + 3 < m) {
          // both halves of every lane inside the matrix: optima tracked per 4 steps
          int hk[4][2];
          step(t0, vh.x, ve.x, vc.x, std::false_type(), hk[0]);
          step(t0 + 1, vh.y, ve.y, vc.y, std::false_type(), hk[1]);
          step(t0 + 2, vh.z, ve.z, vc.z, std::false_type(), hk[2]);
          step(t0 + 3, vh.w, ve.w, vc.w, std::false_type(), hk[3]);
          int mk[2];
          bool imp = false;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            mk[r] = pmax(pmax(hk[0][r], hk[1][r]), pmax(hk[2][r], hk[3][r]));
            imp |= pmax(mk[r], bvr[r]) != bvr[r];
          }
          if (imp) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                auto half = [&](int x) { return h ? hi16(x) : lo16(x); };
                const int mv = half(mk[r]);
                int k = half(hk[2][r]) == mv ? 2 : 3;
                k = half(hk[1][r]) == mv ? 1 : k;
                k = half(hk[0][r]) == mv ? 0 : k;
                const bool up = mv > half(bvr[r]);
                bjA[h][r] = mask_select(__builtin_amdgcn_ballot_w64(up), t0 - lane + 1 - (h ? D : 0) + k, bjA[h][r]);
                bvA[h][r] = max(bvA[h][r], mv + (h ? B1 : B0));
              }
              bvr[r] = pmax(bvr[r], mk[r]);
            }
          }
        } else {
          step(t0, vh.x, ve.x, vc.x, std::true_type(), nullptr);
          step(t0 + 1, vh.y, ve.y, vc.y, std::true_type(), nullptr);
          step(t0 + 2, vh.z, ve.z, vc.z, std::true_type(), nullptr);
          step(t0 + 3, vh.w, ve.w, vc.w, std::true_type(), nullptr);
        }
      }
      // lanes 64-BLK.. hold lane 63's outputs of steps tb..tb+BLK-1: the upper half's bottom row at
      // columns step - 62 (kept for the lower half) and the band's bottom row at step - 62 - D
      const int so = tb + (lane - (64 - BLK));
      const bool inw = lane >= 64 - BLK;
      const int cu = so - 62, cl = so - 62 - D;
      if (inw && cu >= 1 && cu <= m) dl[cu % kDelayRing] = make_int2(unrel16(lo16(out_h), B0), unrel16(lo16(out_e), B0));
      if (has_out) {
        const int hi = min(tb + BLK - 63 - D, m);
        if (hi >= 1) {
          if (!lds_wait_ge(&con[wib + 1], hi - kRing)) {  // the band below has read what this overwrites
            failed = true;
            break;
          }
          if (inw && cl >= 1 && cl <= m) {
            rout_h[(cl - 1) % kRing] = unrel16(hi16(out_h), B1);
            rout_e[(cl - 1) % kRing] = unrel16(hi16(out_e), B1);
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (lane == 0) __hip_atomic_store(&pub[wib + 1], hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }

    // band optimum: (score, i, j) over this lane's rows, then across the wave
    int bs = kNeg32, bi = 0, bjj = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int i = i0 + h * HB + 2 * lane + r + 1;
        if (i > n) continue;
        const int sc = bvA[h][r] + i * ge;
        const int jj = bjA[h][r];
        const int ci = flip ? jj : i, cj = flip ? i : jj;
        if (sc > 0 && better(sc, ci, cj, bs, bi, bjj)) {
          bs = sc;
          bi = ci;
          bjj = cj;
        }
      }
    for (int o = 32; o >= 1; o >>= 1) {
      const int s2_ = __shfl_xor(bs, o, 64), i2 = __shfl_xor(bi, o, 64), j2 = __shfl_xor(bjj, o, 64);
      if (better(s2_, i2, j2, bs, bi, bjj)) {
        bs = s2_;
        bi = i2;
        bjj = j2;
      }
    }
    const bool anybad = __any(bad);
    if (lane == 0) W.band_res[t] = make_int4(bs, bi, bjj, (anybad ? 1 : 0) | (failed ? 2 : 0));
  };

  for (;;) {
    if (threadIdx.x == 0) {
      s_t0 = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(W.ticket), (unsigned long long)kWfWavesPerBlock);
      for (int k = 0; k <= kWfWavesPerBlock; ++k) {
        pub[k] = 0;
        con[k] = 0;
      }
      s_err = 0;
    }
    __syncthreads();
    const int64_t t0g = s_t0;
    if (t0g >= n_items) break;  // the same for the whole workgroup
    const bool launch_err = __hip_atomic_load(W.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    if (!launch_err && wib == kWfWavesPerBlock) {
      courier(t0g);
    } else if (!launch_err && t0g + wib < n_items) {
    if constexpr (P16) {
      p16_band(t0g + wib);
    } else {
    const int64_t t = t0g + wib;
    const WfPair pr = W.pairs[np == 1 ? 0 : W.item_pair[t]];
    const int b = __builtin_amdgcn_readfirstlane((int)(t - pr.item0));
    const int n = __builtin_amdgcn_readfirstlane(pr.n), m = __builtin_amdgcn_readfirstlane(pr.m);
    const int nb = __builtin_amdgcn_readfirstlane(pr.nb);
    // rows come from the query array, columns from the subject array, or the reverse when flipped
    const bool flip = __builtin_amdgcn_readfirstlane(pr.flip) != 0;
    const uint8_t* __restrict__ q = (flip ? S : Q) + pr.q_off;
    const uint8_t* __restrict__ s = (flip ? Q : S) + pr.s_off;

    const int i0 = b * BH, irow0 = i0 + lane * R;
    uint32_t* __restrict__ lp = lprof + (lane_words(PROF) ? cw * (P.alphabet + 1) * 64 + lane : 0);
    LetterWindow<BLK>& lett = letters[cw];
    int prof[R];
    BandLane<R> L;
    BandBest<R> B;
    bool bad = false;
    band_start<MODE, PROF, FA, R>(P, sig2, q, n, flip, irow0, lane, lp, prof, L, B, bad);
    uint16_t* __restrict__ codes = TB ? W.codes + pr.code_off + (size_t)(b * 64 + lane) * (size_t)m : nullptr;
    const bool last_band = (b == nb - 1);
    if (MODE == ALN_SEMIGLOBAL && last_band) last_row_start<R>(P, n - 1 - irow0, B);
    bool failed = false;
    int *rin_h = ring_h(cw), *rin_e = ring_e(cw);           // row of the band above (b > 0)
    int *rout_h = ring_h(cw + 1), *rout_e = ring_e(cw + 1);  // this band's bottom row, for the band below
    const bool has_out = b + 1 < nb;
    // The letters of columns tb - 31 .. tb + 32 are loaded one block ahead and turned into profile indices only when
    // their block starts, so the load's latency hides behind a block of steps; -1 outside the subject.
    auto letter_at = [&](int col) -> int { return col >= 1 && col <= m ? (int)s[col - 1] : -1; };
    int c_next = letter_at(lane - 31);
    int c_idx = letter_index<PROF, R>(P, -1, flip, bad);
    lett.clear_tail(lane);

    const int steps = m + 64;  // lane 63's column m leaves at step m + 63
    for (int tb = 0; tb < steps; tb += BLK) {
      const int col_in = tb + 1 + lane;
      static_assert(BLK == 32, "a wave's lanes hold the letters of two blocks");
      const int c_old = c_idx;  // columns tb - 63 .. tb
      c_idx = letter_index<PROF, R>(P, c_next, flip, bad);
      // consume the previous block's load before issuing the next one: memory counters drain in order,
      // so waiting for the old letter must not also wait for the new load
      asm volatile("" ::"v"(c_idx) : "memory");
      c_next = letter_at(tb + 1 + lane);  // columns (tb + 32) - 31 ..
      lett.v[lane] = c_old;
      if (lane >= 32) lett.v[32 + lane] = c_idx;  // columns tb + 1 .. tb + 32
      const int hi = tb + BLK - 64;  // columns the block's outputs complete (the last ones may lie past m)
      // the band below has read what this block's outputs overwrite
      if (has_out && !lds_wait_ge(&con[cw + 1], hi - kRing)) {
        failed = true;
        break;
      }
      const int need = min(tb + BLK, m);
      int32_t th = lane_neg<FA>();
      if (b == 0) {
        // the ring above is nobody's: this band writes row 0 there itself
        if (lane < BLK) {
          th = border_h<MODE, FA>(P, 0, col_in);
          rin_h[(col_in - 1) % kRing] = th;
          rin_e[(col_in - 1) % kRing] = lane_neg<FA>();
        }
      } else {
        if (!lds_wait_ge(&pub[cw], need)) {
          failed = true;
          break;
        }
        if (lane < BLK && col_in <= m) th = rin_h[(col_in - 1) % kRing];
      }
      if (MODE == ALN_LOCAL)
        B.floor = raise_local_floor(B.bs, lane < BLK && col_in <= m ? th - lane_zero<FA>() + (i0 + col_in) * P.ge : 0);
      auto load_rows = [&](int g4, BandIn<R>& I) __attribute__((always_inline)) {
        const int k = ((tb + 4 * g4) & (kRing - 1)) / 4;
        const int4 h4 = reinterpret_cast<const int4*>(rin_h)[k];
        const int4 e4 = reinterpret_cast<const int4*>(rin_e)[k];
        I.vh[0] = h4.x, I.vh[1] = h4.y, I.vh[2] = h4.z, I.vh[3] = h4.w;
        I.ve[0] = e4.x, I.ve[1] = e4.y, I.ve[2] = e4.z, I.ve[3] = e4.w;
      };
      auto run = [&](int g4, BandIn<R>& I) __attribute__((always_inline)) {
        const int t0 = tb + 4 * g4;
        const int j0 = t0 - lane + 1;
        if (t0 + 4 > m) {
          // past the last column the ring holds whatever it held: nothing above lane 0 there
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            I.vh[u] = t0 + u + 1 > m ? lane_neg<FA>() : I.vh[u];
            I.ve[u] = t0 + u + 1 > m ? lane_neg<FA>() : I.ve[u];
          }
        }
        const int ph = L.bot_h, pe = L.bot_e, floor0 = L.floor0;
        BandGroup<R> G;
        const bool inside = t0 >= 63 && t0 + 3 < m;
        // With checkpoints, some lane's column in these 4 steps is a multiple of kTileCols only when
        // (t0 + 1) mod kTileCols is below 64 or within 3 of kTileCols (a wave-uniform test).
        const int cu = (t0 + 1) & (kTileCols - 1);
        if (CKPT && (cu < 64 || cu > kTileCols - 4)) {
          auto checkpoint = [&](int u) {
            const int j = j0 + u;
            if ((j & (kTileCols - 1)) == 0 && j >= kTileCols && j < m) {
              // rows irow0+1..irow0+4 of column j: H~ and F~, 32 contiguous bytes
              int4* dst = reinterpret_cast<int4*>(W.ckcols + (int64_t)(j / kTileCols - 1) * W.ck_ld + irow0);
              dst[0] = make_int4(L.h[0], L.f[0], L.h[1], L.f[1]);
              dst[1] = make_int4(L.h[2], L.f[2], L.h[3], L.f[3]);
            }
          };
          if (MODE == ALN_LOCAL || t0 >= 63)
            band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupInside>(P, tab, prof, I, j0, m, L, G, checkpoint);
          else
            band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupStart>(P, tab, prof, I, j0, m, L, G, checkpoint);
        } else if (MODE == ALN_LOCAL || t0 >= 63) {
          band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupInside>(P, tab, prof, I, j0, m, L, G, [](int) {});
        } else {
          band_group<MODE, AFFINE, PROF, TB, FA, R, kGroupStart>(P, tab, prof, I, j0, m, L, G, [](int) {});
        }
        if (MODE != ALN_LOCAL && t0 + 4 >= m)
          track_last_column<FA, R, MODE == ALN_GLOBAL>(P, G, j0, n, m, irow0, B);
        if (TB) store_codes<R>(G, codes, j0, m, inside);
        if constexpr (MODE == ALN_LOCAL) track_local<AFFINE, R>(P, L, G, floor0, j0, flip, B);
        if (MODE == ALN_SEMIGLOBAL && last_band) track_last_row<AFFINE, R>(P, L, G, floor0, m, n - 1 - i0, j0, B);
        if (has_out && lane == 63) {
          reinterpret_cast<int4*>(rout_h)[((t0 - 64) & (kRing - 1)) / 4] = make_int4(ph, G.oh[0], G.oh[1], G.oh[2]);
          reinterpret_cast<int4*>(rout_e)[((t0 - 64) & (kRing - 1)) / 4] = make_int4(pe, G.oe[0], G.oe[1], G.oe[2]);
        }
      };
      run_block<PROF, R, BLK / 4, WAVES < 5>(lett, lp, lane, min(BLK / 4, (steps - tb + 3) / 4), load_rows, run);
      // the block's ring reads are complete and its outputs written before either is announced
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (lane == 0) {
        if (b > 0) __hip_atomic_store(&con[cw], need, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (has_out && hi >= 1)
          __hip_atomic_store(&pub[cw + 1], min(hi, m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    const int4 opt = band_optimum<MODE, FA, R>(P, B, n, m, flip, last_band, irow0, bad, failed);
    if (lane == 0) W.band_res[t] = opt;
    }
    }
    __syncthreads();  // the group's rings and ticket are reused by the next group
  }
}

// A pair's result from its bands' optimum (bs at bi, bj) and flags, without the traceback's part.
__device__ __forceinline__ aln_result_t pair_result(const KParams& P, const WfPair& pr, int bs, int bi, int bj, int flag,
                                                    bool err) {
  const int n = pr.flip ? pr.m : pr.n, m = pr.flip ? pr.n : pr.m;  // the call's query and subject lengths
  aln_result_t r;
  r.q_begin = -1;
  r.s_begin = -1;
  r.cigar_len = 0;
  r.reserved = 0;
  r.flags = 0;
  if (P.mode == ALN_GLOBAL) {
    r.q_end = n;
    r.s_end = m;
    r.score = (n == 0 || m == 0) ? ((n + m > 0) ? P.go + (n + m) * P.ge : 0) : bs;
  } else if (n == 0 || m == 0 || bs < 0 || (bs == 0 && P.mode == ALN_LOCAL)) {
    // local: the empty alignment at (0,0); semi-global: the first candidate (0, m), or (0, 0) if a side is empty
    r.score = 0;
    r.q_end = 0;
    r.s_end = (P.mode == ALN_SEMIGLOBAL && n > 0) ? m : 0;
  } else if (P.mode == ALN_SEMIGLOBAL && bs == 0) {
    r.score = 0;  // (0, m) precedes every other candidate in row-major order
    r.q_end = 0;
    r.s_end = m;
  } else {
    r.score = bs;
    r.q_end = bi;
    r.s_end = bj;
  }
  if (err || (flag & 2)) r.flags |= ALN_RES_DEVICE_ERROR;
  if (flag & 1) {
    r.flags |= ALN_RES_BAD_CODE;
    r.score = 0;
    r.q_end = 0;
    r.s_end = 0;
  }
  return r;
}

// Reduces every pair's band optima into its aln_result_t.  A wave takes as many consecutive pairs as spread the batch
// over the launch's waves, up to 64: its lanes finish one pair with one band each (100,003 of them took 113 us with a
// wave each), and the whole wave takes the other pairs one at a time.
// cigar_off, when given, is a batch call's: pair out_idx owns cigar[cigar_off[out_idx] .. cigar_off[out_idx + 1]];
// otherwise the single pair owns cigar_cap words at cigar.
template <int MODE, bool TB>
__global__ __launch_bounds__(256) void wf_finish_kernel(const KParams P, WfWs W, const uint8_t* __restrict__ q,
                                                        const uint8_t* __restrict__ s,
                                                        aln_result_t* __restrict__ out,
                                                        uint32_t* __restrict__ cigar, int64_t cigar_cap,
                                                        const int64_t* __restrict__ cigar_off) {
  __shared__ uint16_t walk_win[TB ? 4 : 1][TB ? kWalkCodes : 1];
  const int lane = threadIdx.x & 63;
  const int np = *W.n_pairs;
  const int waves = (int)gridDim.x * 4;
  const int per = TB ? 1 : min(64, max(1, np / waves));
  const bool err = __hip_atomic_load(W.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  for (int64_t k0 = (int64_t)(blockIdx.x * 4 + (threadIdx.x >> 6)) * per; k0 < np; k0 += (int64_t)waves * per) {
    unsigned long long rest = per == 64 ? ~0ull : (1ull << per) - 1;  // pairs left to the whole wave
    if (per > 1) {
      bool left = false;
      if (lane < per && k0 + lane < np) {
        const WfPair pr = W.pairs[k0 + lane];
        left = pr.nb != 1;
        if (!left) {
          const int4 v = W.band_res[pr.item0];
          out[pr.out_idx] = pair_result(P, pr, v.x, v.y, v.z, v.w, err);
        }
      }
      rest = __builtin_amdgcn_ballot_w64(left);
    }
    for (; rest; rest &= rest - 1) {
      const int64_t k = k0 + __builtin_ctzll(rest);
      const WfPair pr = W.pairs[k];
      int bs = kNeg32, bi = 0, bj = 0, flag = 0;
      for (int b = lane; b < pr.nb; b += 64) {
        const int4 v = W.band_res[pr.item0 + b];
        flag |= v.w;
        if (better(v.x, v.y, v.z, bs, bi, bj)) {
          bs = v.x;
          bi = v.y;
          bj = v.z;
        }
      }
      if (pr.nb == 0) {
        // a pair with an empty side has no bands, whose relaxation checks the letters: check them here
        const uint8_t* rq = (pr.flip ? s : q) + pr.q_off;  // the pair's row and column letters
        const uint8_t* rs = (pr.flip ? q : s) + pr.s_off;
        for (int c = lane; c < pr.n; c += 64)
          if (rq[c] >= P.alphabet) flag |= 1;
        for (int c = lane; c < pr.m; c += 64)
          if (rs[c] >= P.alphabet) flag |= 1;
      }
      for (int o = 32; o >= 1; o >>= 1) {
        const int s2 = __shfl_xor(bs, o, 64), i2 = __shfl_xor(bi, o, 64), j2 = __shfl_xor(bj, o, 64);
        flag |= __shfl_xor(flag, o, 64);
        if (better(s2, i2, j2, bs, bi, bj)) {
          bs = s2;
          bi = i2;
          bj = j2;
        }
      }
      // every lane now holds the same optimum; the result is computed by all and written by lane 0
      aln_result_t r = pair_result(P, pr, bs, bi, bj, flag, err);
      if (TB && r.flags == 0) {
        // The codes form a [row group][column] array of 16-bit words, 4 rows per word (band bb, lane L
        // is row group bb * 64 + L); walk_core walks them with the whole wave.
        uint32_t* cg = cigar;
        int64_t cap = cigar_cap;
        if (cigar_off) {
          const int64_t c0 = cigar_off[pr.out_idx];
          cg = cigar + c0;
          cap = cigar_off[pr.out_idx + 1] - c0;
        }
        WalkState S;
        walk_start(S, r.q_end, r.s_end);
        walk_core<MODE>(W.codes + pr.code_off, pr.m, 0, 0, 0, S, walk_win[threadIdx.x >> 6], lane, cg, cap);
        const int64_t runs = walk_finish(S, lane, cg, cap);
        r.q_begin = S.i;
        r.s_begin = S.j;
        r.cigar_len = (int)runs;
        if (runs > cap) r.flags |= ALN_RES_CIGAR_TRUNC;
        if (S.stuck) r.flags |= ALN_RES_DEVICE_ERROR;
      }
      if (lane == 0) out[pr.out_idx] = r;
    }
  }
}

// Before a wavefront launch: clears the progress counter of every item and the ticket, and maps
// every item to its pair.
__global__ void wf_reset_kernel(WfWs W) {
  const int64_t n_items = *W.n_items;
  const int np = *W.n_pairs;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n_items; k += stride) W.flags[k] = 0;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < 2 * (int64_t)W.n_lv - 1; k += stride)
    W.lv[k] = 0;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < np; k += stride) {
    const WfPair pr = W.pairs[k];
    for (int b = 0; b < pr.nb; ++b) W.item_pair[pr.item0 + b] = (int)k;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *W.ticket = 0;
    *W.error = 0;
  }
}

// The order in which the per-band engine hands out its items: level by level, band 0 of every pair
// (in the planner's order, largest band work first), then band 1 of every pair, and so on.  Pair-major
// order handed out all the bands of a pair at once, and band b then waited about b lags for the bands
// above it, idle -- a fifth of the waves' time on square pairs, whatever their size -- while other
// pairs' bands could have run.  Level by level, a band is handed out only after every band of the
// level above, so band b - 1 of its pair is always already running (no deadlock, whatever the
// residency) and usually far ahead.  On the uneven protein batch this took the call from 250 to 175 ms;
// chunks of 64 to 16384 pairs ordered this way, one chunk after the other, gave 230 to 177.
//
// W.lv: [0] the largest band count, [1 .. L] the pairs with exactly b bands, then the first position
// of level b, [L + 1 ..] the level cursors (L = W.n_lv - 1 entries each, cleared by wf_reset_kernel).
__global__ __launch_bounds__(256) void wf_level_hist_kernel(WfWs W) {
  const int np = *W.n_pairs;
  const int L = W.n_lv - 1;
  const int lane = threadIdx.x & 63;
  int mx = 0;
  for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); p0 < np;
       p0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = p0 + lane;
    const int nb = p < np ? W.pairs[p].nb : 0;
    mx = max(mx, nb);
    // one atomic per distinct band count among the wave's pairs (the planner's order keeps them few)
    bool left = nb > 0 && nb <= L;
    while (__builtin_amdgcn_ballot_w64(left) != 0) {
      const unsigned long long lm = __builtin_amdgcn_ballot_w64(left);
      const int first = (int)__builtin_ctzll(lm);
      const int v = __shfl(nb, first, 64);
      const bool same = left && nb == v;
      const unsigned long long sm = __builtin_amdgcn_ballot_w64(same);
      if (lane == first) atomicAdd(&W.lv[v], (int)__builtin_popcountll(sm));
      left = left && !same;
    }
  }
  mx = __ockl_wfred_max_i32(mx);
  if (lane == 0 && mx > 0) atomicMax(&W.lv[0], min(mx, L));
}

// One block: level b holds the pairs with more than b bands; its items start after those of levels
// 0 .. b - 1.  Overwrites the histogram with the first position of every level.
__global__ __launch_bounds__(1024) void wf_level_scan_kernel(WfWs W) {
  __shared__ int64_t part[1024];
  const int L = min(W.lv[0], W.n_lv - 1);
  // cnt(b) = pairs with more than b bands = sum of hist[h], h > b; then the exclusive prefix of cnt
  int64_t run_cnt = 0;  // pairs with more than the current chunk's bands (suffix sum so far)
  // levels in chunks of 1024, from the top: cnt needs a suffix sum over the histogram
  const int chunks = (L + 1023) / 1024;
  // pass 1: cnt(b) in place of hist(b + 1) (hist(b + 1) is read before it is overwritten)
  for (int c = chunks - 1; c >= 0; --c) {
    const int b = c * 1024 + threadIdx.x;  // level b counts hist[b + 1 .. L]
    const int64_t h = (b < L) ? (int64_t)W.lv[b + 1] : 0;
    part[threadIdx.x] = h;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {  // suffix sums within the chunk
      const int64_t a = threadIdx.x + o < 1024 ? part[threadIdx.x + o] : 0;
      __syncthreads();
      part[threadIdx.x] += a;
      __syncthreads();
    }
    const int64_t cnt = part[threadIdx.x] + run_cnt;
    const int64_t chunk_total = part[0];
    __syncthreads();
    if (b < L) W.lv[b + 1] = (int)cnt;  // now cnt(b) at lv[b + 1]
    run_cnt += chunk_total;
    __syncthreads();
  }
  // pass 2: exclusive prefix of cnt over the levels: the first position of level b, at lv[b + 1]
  int64_t run = 0;
  for (int c = 0; c < chunks; ++c) {
    const int b = c * 1024 + threadIdx.x;
    const int64_t v = (b < L) ? (int64_t)W.lv[b + 1] : 0;
    part[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int64_t a = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
      __syncthreads();
      part[threadIdx.x] += a;
      __syncthreads();
    }
    const int64_t incl = part[threadIdx.x];
    const int64_t total = part[1023];
    __syncthreads();
    if (b < L) W.lv[b + 1] = (int)(run + incl - v);
    run += total;
    __syncthreads();
  }
}

// One wave per 64 consecutive pairs: each level's items of the wave's pairs get consecutive positions
// from the level's cursor, in pair order.
__global__ __launch_bounds__(256) void wf_order_kernel(WfWs W) {
  const int np = *W.n_pairs;
  const int L = W.n_lv - 1;
  const int lane = threadIdx.x & 63;
  const int64_t nchunks = ((int64_t)np + 63) / 64;
  const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
  const int64_t waves = (int64_t)gridDim.x * blockDim.x / 64;
  int* cur = W.lv + 1 + L;
  for (int64_t c = wave0; c < nchunks; c += waves) {
    const int64_t p = c * 64 + lane;
    int nb = 0;
    int64_t it0 = 0;
    if (p < np) {
      const WfPair pr = W.pairs[p];
      nb = pr.nb <= L ? pr.nb : 0;
      it0 = pr.item0;
    }
    const int wmax = __ockl_wfred_max_i32(nb);
    // 64 levels at a time: lane u counts the wave's pairs at level b0 + u, reserves their places with one
    // atomic (all lanes' atomics in one instruction) and reads the level's first position
    for (int b0 = 0; b0 < wmax; b0 += 64) {
      const int nl = min(64, wmax - b0);
      int mycnt = 0;
      for (int u = 0; u < nl; ++u) {
        const int cnt = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(b0 + u < nb));
        if (lane == u) mycnt = cnt;
      }
      int mybase = 0;
      if (lane < nl && mycnt > 0) mybase = W.lv[1 + b0 + lane] + atomicAdd(&cur[b0 + lane], mycnt);
      for (int u = 0; u < nl; ++u) {
        const int b = b0 + u;
        const bool has = b < nb;
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(has);
        const int at = __shfl(mybase, u, 64);
        const int rank = (int)__builtin_popcountll(mask & ((1ull << lane) - 1ull));
        if (has) W.order[(int64_t)at + rank] = it0 + b;
      }
    }
  }
}

// align_long: describes the single pair as the only entry of the pair table.
__global__ void wf_single_pair_kernel(WfWs W, int n, int m, int band_rows) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    WfPair p;
    p.q_off = 0;
    p.s_off = 0;
    p.n = n;
    p.m = m;
    p.nb = (n > 0 && m > 0) ? (n + band_rows - 1) / band_rows : 0;
    p.item0 = 0;
    p.row_off = 0;
    p.code_off = 0;
    p.out_idx = 0;
    p.flip = 0;
    p.pad_ = 0;
    W.pairs[0] = p;
    *W.n_pairs = 1;
    *W.n_items = p.nb;
  }
}

// Packed 16-bit bands are exact when a block's scores stay within int16 of its offsets: a block's
// cells lie within 128 rows and 63 + 32 columns of the offset's cell, and the block's own 32 steps
// move the offset's column by at most 32 more; adjacent cells differ by at most max|sigma| + |go| +
// 2|ge| (row bias included), and E, F lie within |go + ge| of a neighbouring H.  Bounding that step
// by 32 keeps every value of a block within (128 + 95 + 32) x 32 = 8,160 of its offset, far from the
// -32,768 that stands for -infinity.
bool p16_exact(const KParams& kp) {
  const int64_t smax = kp.sigma_max > -kp.sigma_min ? kp.sigma_max : -(int64_t)kp.sigma_min;
  const int64_t step = smax - kp.go - 2 * (int64_t)kp.ge;
  return step <= 32;
}

template <int MODE, bool AFFINE, int PROF, bool TB, bool FA>
void launch_wf_t(const KParams& kp, const uint8_t* q, const uint8_t* s, const WfWs& W, int n_waves, bool grouped,
                 bool crowded, bool p16, hipStream_t stream) {
  const int blocks = (n_waves + kWfWavesPerBlock - 1) / kWfWavesPerBlock;
  const size_t lds = lane_words(PROF) ? (size_t)kWfWavesPerBlock * (kp.alphabet + 1) * 64 * sizeof(uint32_t) : 0;
  constexpr bool kCanPack = MODE == ALN_LOCAL && (PROF == kProfReg || PROF == kProfLane) && !TB;
  if (kCanPack && grouped && p16 && p16_exact(kp)) {
    // packed bands keep two 16-bit rows of each half per letter and lane: twice the words
    ProfScope prof("wavefront_p16", stream);
    hipLaunchKernelGGL((wf_i32_group_kernel<MODE, AFFINE, PROF, TB, false, kWfR, kCanPack, false, 4>), dim3(blocks),
                       dim3(kWfBlock), 2 * lds, stream, kp, q, s, W);
    return;
  }
  // Local linear score-only bands in groups: their steps wait for latency (30000 x 30000 5.03 and 4.68 ms), where bands on their own
  // fill the SIMD and the dot product's fewer issue slots are worth more (1500 pairs of 2000..6000 4.48 and 4.86).
  constexpr int kGroupProf = PROF == kProfReg && MODE == ALN_LOCAL && !AFFINE && !TB ? kProfRegBits : PROF;
  if constexpr (!TB) {
    if (W.ckcols) {
      ProfScope prof("wavefront_i32_checkpoints", stream);
      hipLaunchKernelGGL((wf_i32_group_kernel<MODE, AFFINE, kGroupProf, TB, FA, kWfR, false, true, 3>), dim3(blocks),
                         dim3(kWfBlock), lds, stream, kp, q, s, W);
      return;
    }
  }
  ProfScope prof(TB ? "wavefront_i32_traceback" : "wavefront_i32", stream);
  if (grouped) {
    if constexpr (!TB) {
      if (crowded) {
        hipLaunchKernelGGL((wf_i32_group_kernel<MODE, AFFINE, kGroupProf, TB, FA, kWfR, false, false, 5>), dim3(blocks),
                           dim3(kWfBlock), lds, stream, kp, q, s, W);
        return;
      }
    }
    hipLaunchKernelGGL((wf_i32_group_kernel<MODE, AFFINE, kGroupProf, TB, FA, kWfR, false, false, 4>), dim3(blocks),
                       dim3(kWfBlock), lds, stream, kp, q, s, W);
  } else
    hipLaunchKernelGGL((wf_i32_kernel<MODE, AFFINE, PROF, TB, FA, kWfR>), dim3(blocks), dim3(kWfBlockAlone), lds,
                       stream, kp, q, s, W);
}

template <int MODE, bool AFFINE, bool TB, bool FA>
void launch_wf_p(const KParams& kp, const uint8_t* q, const uint8_t* s, const WfWs& W, int nw, bool grouped, bool crowded, bool p16,
                 hipStream_t st) {
  const bool bytes = score_bytes(kp), lowered = lowered_score_bytes(kp);
  if (bytes && kp.alphabet <= 4)
    launch_wf_t<MODE, AFFINE, kProfReg, TB, FA>(kp, q, s, W, nw, grouped, crowded, p16, st);
  else if (lowered && kp.alphabet <= 4)
    launch_wf_t<MODE, AFFINE, kProfRegLow, TB, FA>(kp, q, s, W, nw, grouped, crowded, false, st);
  else if (bytes)
    launch_wf_t<MODE, AFFINE, kProfLane, TB, FA>(kp, q, s, W, nw, grouped, crowded, p16, st);
  else if (lowered && kp.sig_off <= 127)  // (128 and more would lift the pad letter's -128 above 0)
    launch_wf_t<MODE, AFFINE, kProfLaneLow, TB, FA>(kp, q, s, W, nw, grouped, crowded, false, st);
  else
    launch_wf_t<MODE, AFFINE, kProfTable, TB, FA>(kp, q, s, W, nw, grouped, crowded, false, st);
}

// fa: float lanes (band.h).  Only affine gaps add a constant per cell; linear ones always use integer lanes.
template <int MODE, bool TB>
void launch_wf_m(const KParams& kp, const uint8_t* q, const uint8_t* s, const WfWs& W, int nw, bool grouped, bool crowded, bool p16,
                 bool fa, hipStream_t st) {
  if (kp.go == 0)
    launch_wf_p<MODE, false, TB, false>(kp, q, s, W, nw, grouped, crowded, p16, st);
  else if (fa)
    launch_wf_p<MODE, true, TB, true>(kp, q, s, W, nw, grouped, crowded, p16, st);
  else
    launch_wf_p<MODE, true, TB, false>(kp, q, s, W, nw, grouped, crowded, p16, st);
}

template <int MODE>
void launch_wf_mode(const KParams& kp, const uint8_t* q, const uint8_t* s, const WfWs& W, int nw, bool grouped, bool crowded,
                    bool tb, bool p16, bool fa, aln_result_t* out, uint32_t* cigar, int64_t cap, const int64_t* cigar_off,
                    hipStream_t st) {
  if (tb) {
    launch_wf_m<MODE, true>(kp, q, s, W, nw, grouped, false, false, fa, st);
    hipLaunchKernelGGL((wf_finish_kernel<MODE, true>), dim3(256), dim3(256), 0, st, kp, W, q, s, out, cigar, cap,
                       cigar_off);
  } else {
    launch_wf_m<MODE, false>(kp, q, s, W, nw, grouped, crowded, p16, fa, st);
    hipLaunchKernelGGL((wf_finish_kernel<MODE, false>), dim3(256), dim3(256), 0, st, kp, W, q, s, out, cigar, cap,
                       cigar_off);
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

bool band_fits_fa(const KParams& kp, int64_t n, int64_t m) {
  const int64_t c = -(int64_t)kp.ge, mn = n < m ? n : m;
  const int64_t up = mn * (kp.sigma_max > 0 ? kp.sigma_max : 0) + (n + m + 2 * kWfBand) * c + 256;
  const int64_t down = 64 * c - 4 * (int64_t)kp.go + 256;  // columns before the first; gaps opened from there
  return up < (1 << 23) - (1 << 20) && down < (1 << 20);
}

int wf_waves(int per_cu) {
  const int cus = device_cu_count();
  if (per_cu < 1 || per_cu > kWfWavesPerCUMax) return -1;
  return cus > 0 ? cus * per_cu : -1;
}

size_t wf_layout(int64_t max_pairs, int64_t max_items, int64_t row_words, int64_t code_words, WfOffsets* o) {
  size_t off = 0;
  o->pairs = off;
  off += align256((size_t)max_pairs * sizeof(WfPair));
  o->rows = off;
  off += align256((size_t)row_words * sizeof(int2));
  o->flags = off;
  off += align256((size_t)(max_items + 1) * sizeof(int));
  o->item_pair = off;
  off += align256((size_t)(max_items + 1) * sizeof(int));
  o->res = off;
  off += align256((size_t)(max_items + 1) * sizeof(int4));
  o->misc = off;
  off += 256;
  o->codes = off;
  off += align256((size_t)code_words * sizeof(uint16_t));
  o->order = off;
  off += align256((size_t)(max_items + 1) * sizeof(int64_t));
  // a pair has at most max_items bands
  o->n_lv = max_items + 2;
  o->lv = off;
  off += align256((size_t)(2 * o->n_lv - 1) * sizeof(int));
  return off;
}

WfWs wf_view(void* base_, const WfOffsets& o) {
  char* base = static_cast<char*>(base_);
  WfWs W;
  W.pairs = reinterpret_cast<WfPair*>(base + o.pairs);
  W.rows = reinterpret_cast<int2*>(base + o.rows);
  W.flags = reinterpret_cast<int*>(base + o.flags);
  W.item_pair = reinterpret_cast<int*>(base + o.item_pair);
  W.band_res = reinterpret_cast<int4*>(base + o.res);
  W.ticket = reinterpret_cast<int64_t*>(base + o.misc);
  W.n_items = reinterpret_cast<int64_t*>(base + o.misc + 8);
  W.n_pairs = reinterpret_cast<int*>(base + o.misc + 16);
  W.error = reinterpret_cast<int*>(base + o.misc + 20);
  W.codes = reinterpret_cast<uint16_t*>(base + o.codes);
  W.ckcols = nullptr;
  W.ck_ld = 0;
  W.order = reinterpret_cast<int64_t*>(base + o.order);
  W.lv = reinterpret_cast<int*>(base + o.lv);
  W.n_lv = (int)o.n_lv;
  return W;
}

aln_status_t launch_wf_i32(const KParams& kp, const WfWs& W, const uint8_t* q, const uint8_t* s,
                           aln_result_t* out, int max_waves, bool grouped, bool crowded, bool tb, bool p16, bool fa, uint32_t* cigar,
                           int64_t cigar_cap, hipStream_t stream, const int64_t* cigar_off) {
  hipLaunchKernelGGL(wf_reset_kernel, dim3(256), dim3(256), 0, stream, W);
  if (!grouped) {
    hipLaunchKernelGGL(wf_level_hist_kernel, dim3(256), dim3(256), 0, stream, W);
    hipLaunchKernelGGL(wf_level_scan_kernel, dim3(1), dim3(1024), 0, stream, W);
    hipLaunchKernelGGL(wf_order_kernel, dim3(256), dim3(256), 0, stream, W);
  }
  switch (kp.mode) {
    case ALN_GLOBAL:
      launch_wf_mode<ALN_GLOBAL>(kp, q, s, W, max_waves, grouped, crowded, tb, p16, fa, out, cigar, cigar_cap, cigar_off, stream);
      break;
    case ALN_LOCAL:
      launch_wf_mode<ALN_LOCAL>(kp, q, s, W, max_waves, grouped, crowded, tb, p16, fa, out, cigar, cigar_cap, cigar_off, stream);
      break;
    default:
      launch_wf_mode<ALN_SEMIGLOBAL>(kp, q, s, W, max_waves, grouped, crowded, tb, p16, fa, out, cigar, cigar_cap, cigar_off,
                                     stream);
      break;
  }
  return hipGetLastError() == hipSuccess ? ALN_OK : ALN_E_DEVICE;
}

// ---------------------------------------------------------------------------------------------
// aln_align_long: the engine on one pair.
// ---------------------------------------------------------------------------------------------
aln_status_t plan_long(int64_t n, int64_t m, bool tb, LongPlan* pl) {
  pl->nb = (n + kWfBand - 1) / kWfBand;
  pl->tb = tb;
  const int nw = wf_waves(kWfWavesPerCUDefault);
  if (nw <= 0) return ALN_E_DEVICE;
  int64_t waves = nw;
  const int64_t want = (pl->nb + kWfWavesPerBlock - 1) / kWfWavesPerBlock * kWfWavesPerBlock;
  if (want < waves) waves = want;
  if (waves < kWfWavesPerBlock) waves = kWfWavesPerBlock;
  pl->n_waves = (int)waves;
  const int64_t code_words = tb ? pl->nb * 64 * m : 0;
  pl->total_bytes = wf_layout(1, pl->nb, 2 * (m + 1), code_words, &pl->off);
  return ALN_OK;
}

void launch_single_pair(const WfWs& W, int n, int m, hipStream_t stream) {
  hipLaunchKernelGGL(wf_single_pair_kernel, dim3(1), dim3(64), 0, stream, W, n, m, kWfBand);
}

aln_status_t launch_long(const KParams& kp, const LongPlan& pl, const uint8_t* q, int64_t n, const uint8_t* s,
                         int64_t m, aln_result_t* out, uint32_t* cigar, int64_t cigar_cap, void* ws,
                         hipStream_t stream) {
  WfWs W = wf_view(ws, pl.off);
  hipLaunchKernelGGL(wf_single_pair_kernel, dim3(1), dim3(64), 0, stream, W, (int)n, (int)m, kWfBand);
  // one pair: its bands are few per SIMD, so the grouped engine (no device-memory stalls in the
  // compute waves) is the faster one
  return launch_wf_i32(kp, W, q, s, out, pl.n_waves, true, false, pl.tb, false, band_fits_fa(kp, n, m), cigar,
                       cigar_cap, stream);
}

}  // namespace mialign
