// Row-wise top-k for rows wider than one wavefront's registers can hold (8192 < M <= 65536): one
// workgroup of W wavefronts per row.  Same method as rtopk_kernel.hpp (RTop-K, arXiv 2409.00822,
// Section 3.1, Algorithms 1 and 2); the paper's own kernel stops at M = 8192 (Appendix B), the width its
// shared-memory row buffer allows.  Here every wavefront keeps its slice of the row in VGPRs, and what
// the wavefronts exchange through LDS is small: the slice minima and maxima once, one count per
// wavefront per search step, and one table of per-group candidate counts for the final ranking.
//
// Layout.  Wavefront w, lane l owns NG groups of G consecutive columns:
//   element e = g*G + c  <->  column ((g*W + w)*64 + l)*G + c
// (where the row's end falls inside a lane's group, that lane holds the row's last G columns instead, and
// those of them that the lane before it owns are masked out; see group_col)
// so every load instruction of a wavefront still covers 64*G*4 contiguous bytes, the W wavefronts of a
// group step cover W KiB contiguous, and column order is (g, w, lane, c).  W is 4, 8 or 16, chosen so
// that a lane holds up to 64 values: fewer, fatter wavefronts spread the per-step fixed cost (two
// cross-lane sums, the LDS round trip, the barrier) over more elements, and narrower workgroups leave
// room for more rows per compute unit, whose load and search phases then overlap.
//
// That is rtopk_block_kernel, the full-width search.  rtopk_filter_kernel, which launch_block prefers for small k, searches a
// list of candidates above a floor instead (rtopk_filter.hpp) and comes here only for rows whose list does not hold.
//
// Every wavefront evaluates the same thresholds on the same totals, so all of them take the same
// branches and reach the same barriers; the trip count of the search is uniform over the workgroup.
//
// Template parameters beyond the layout, all with the meaning they have in rtopk_kernel.hpp:
//   MODE (kEarly / kExact / kEps), NEG (the k smallest), DT (fp32, half or bfloat16 rows),
//   DENSE (chosen values in place and zero elsewhere instead of (value, column) pairs; fp32 only).
#pragma once

#include "rtopk_kernel.hpp"

namespace rtopk {

// Inclusive prefix sum over the 64 lanes of a wavefront (not on the hot path: used once per row).
__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int t = __shfl_up(v, d, kWave);
    if (lane >= d) v += t;
  }
  return v;
}

// Sum over each row of 16 lanes; every lane of a row ends up with its row's total.
__device__ __forceinline__ uint32_t row16_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);  // row_half_mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false);  // row_mirror
  return v;
}

// The lane's candidate bits against t: lane_below_packs' layout, set when key >= t.  The same sign-bit
// test as the search's counts, so the set bits of a lane number exactly the keys not counted as below t.
template <int E, bool NEG>
__device__ __forceinline__ void lane_bits_at_or_above(const float (&x)[E], float t, uint32_t (&w)[(E + 31) / 32]) {
  lane_below_packs<E, NEG>(x, t, w);
#pragma unroll
  for (int g = 0; g < (E + 31) / 32; ++g) w[g] = ~w[g] & pack_valid<E>(g);
}

// The G bits of elements g*G .. g*G + G - 1 out of lane_bits_at_or_above's words; element g*G is the
// highest of them.  G divides 32, so a group never straddles two words.
template <int E, int G>
__device__ __forceinline__ uint32_t group_bits(const uint32_t (&w)[(E + 31) / 32], int g) {
  static_assert(32 % G == 0, "a group must not straddle two words");
  const int e0 = g * G, word = e0 / 32;
  const int filled = (word == (E + 31) / 32 - 1 && E % 32 != 0) ? E % 32 : 32;
  return __builtin_amdgcn_ubfe(w[word], (uint32_t)(filled - (e0 % 32) - G), (uint32_t)G);
}

// In the lanes where pos < limit (unsigned; a lane that must not store passes pos = 0xffffffff): the value
// goes to slot pos of vals and col0 + C to slot pos of cols.  The compare leaves its mask in VCC; when
// no lane stores -- the usual case when k is a small part of the row -- one branch skips everything,
// and otherwise the mask becomes the set of active lanes for the address arithmetic and the two
// stores, with no work on the scalar unit beyond saving and restoring that set.
template <int DT, int C>
__device__ __forceinline__ void store_pair_if_below(uint32_t pos, uint32_t limit, void* vals, uint32_t value_bits,
                                                    int32_t* cols, int32_t col0) {
  uint64_t saved;
  uint32_t t1, t2;
  if constexpr (DT == kF32) {
    asm volatile(
        "v_cmp_gt_u32 vcc, %[lim], %[pos]\n\t"
        "s_cbranch_vccz 1f\n\t"
        "s_and_saveexec_b64 %[sv], vcc\n\t"
        "v_lshlrev_b32 %[t1], 2, %[pos]\n\t"
        "v_add_u32 %[t2], %[c], %[col0]\n\t"
        "global_store_dword %[t1], %[val], %[vals]\n\t"
        "global_store_dword %[t1], %[t2], %[cols]\n\t"
        "s_mov_b64 exec, %[sv]\n"
        "1:"
        : [sv] "=&s"(saved), [t1] "=&v"(t1), [t2] "=&v"(t2)
        : [lim] "s"(limit), [pos] "v"(pos), [c] "n"(C), [col0] "v"(col0), [val] "v"(value_bits), [vals] "s"(vals),
          [cols] "s"(cols)
        : "memory", "scc", "vcc");
  } else {
    uint32_t t3;
    asm volatile(
        "v_cmp_gt_u32 vcc, %[lim], %[pos]\n\t"
        "s_cbranch_vccz 1f\n\t"
        "s_and_saveexec_b64 %[sv], vcc\n\t"
        "v_lshlrev_b32 %[t1], 2, %[pos]\n\t"
        "v_lshlrev_b32 %[t3], 1, %[pos]\n\t"
        "v_add_u32 %[t2], %[c], %[col0]\n\t"
        "global_store_short %[t3], %[val], %[vals]\n\t"
        "global_store_dword %[t1], %[t2], %[cols]\n\t"
        "s_mov_b64 exec, %[sv]\n"
        "1:"
        : [sv] "=&s"(saved), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)
        : [lim] "s"(limit), [pos] "v"(pos), [c] "n"(C), [col0] "v"(col0), [val] "v"(value_bits), [vals] "s"(vals),
          [cols] "s"(cols)
        : "memory", "scc", "vcc");
  }
}

// Register budget: a row of 64 values per lane compiles to 83 registers, i.e. 5 wavefronts per SIMD and,
// at 8 wavefronts per workgroup, two rows per compute unit.  Forcing 80 registers (a third row per
// compute unit, at the price of 5 spilled registers) measured no faster in exact mode and 7-15 % slower
// with early stopping, so the allocation is left to the compiler.
// Groups of a row that a workgroup loads ahead, during the ranking of its previous row (16-wavefront
// shape only: the others are launched with one workgroup per row): RTOPK_BLOCK_AHEAD values per lane,
// half of the row, which is what the register budget of four wavefronts per SIMD leaves free.
#ifndef RTOPK_BLOCK_AHEAD
#define RTOPK_BLOCK_AHEAD 32
#endif
// (Measured on 1 GiB inputs: 4096 x 65536 exact 357 us with a workgroup per row, 347 us looping, 319 us with
// 32 values loaded ahead, 324 us with 24, 361 us with 40, which spills.  The narrower shapes, which have two
// to four workgroups on a compute unit whose phases overlap anyway, lose: 8192 x 32768 247 -> 278 us,
// 16384 x 16384 249 -> 299 us when each resident workgroup walks a fixed share of the rows.
// Loading the other half as well, each group of the next row into the registers of the group the ranking
// has just finished with, costs no register on paper but 23 spilled ones in practice: 319 -> 415 us.)
#ifndef RTOPK_BLOCK_PERSIST_MIN_W
#define RTOPK_BLOCK_PERSIST_MIN_W 16
#endif
constexpr bool block_persistent(int W) { return W >= RTOPK_BLOCK_PERSIST_MIN_W; }
// How a row is selected: by the full-width search; through the lists of rtopk_filter.hpp, and by the full-width search
// where they do not hold it; or through the lists alone.
enum BlockPath : int { kFullWidth = 0, kListsFirst = 1, kListsOnly = 2 };
constexpr int block_groups_ahead(int W, int G, int path) { return block_persistent(W) && path == kFullWidth ? RTOPK_BLOCK_AHEAD / G : 0; }

// Groups FIRST .. LAST - 1 of the row of M columns at `from`.  Lanes past M load the row's last columns (in bounds,
// cannot change min or max).
template <int DT, int G, int W, int FIRST, int LAST, int SIZE>
__device__ __forceinline__ void block_load(const typename std::conditional<DT == kF32, float, uint16_t>::type* from, int M,
                                           int lane, int wave, float (&to)[SIZE]) {
  asm volatile("" : "+v"(lane));  // opaque: the columns computed for one row's loads are not kept for the next row's
#pragma unroll
  for (int g = FIRST; g < LAST; ++g) {
    float v[G];
    load_group<DT, G>(from, min(((g * W + wave) * kWave + lane) * G, M - G), v);
#pragma unroll
    for (int c = 0; c < G; ++c) to[g * G + c] = v[c];
  }
}

// Columns past M must never be counted or chosen: their key becomes -inf.
template <int G, int NG, int W, bool NEG>
__device__ __forceinline__ void block_mask(float (&x)[G * NG], int M, int lane, int wave) {
  if (M == kWave * G * NG * W) return;  // uniform: full-width rows skip the masking
  const float none = NEG ? __builtin_inff() : -__builtin_inff();
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if ((g + 1) * (W * kWave * G) <= M) continue;  // uniform: the group lies inside the row
    const int left = M - ((g * W + wave) * kWave + lane) * G;  // columns of the row from the lane's first on
    // past the end, or (M % G != 0) the straddling lane's leading elements, which the lane before it owns
#pragma unroll
    for (int c = 0; c < G; ++c) x[g * G + c] = left < G - c ? none : x[g * G + c];
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Minimum and maximum of the row's keys and, with FILTER, its floor (rtopk_filter.hpp: at least `need` group maxima of
// the wavefront, J per lane, at or above it) and the bound above it: per lane, per wavefront, then over the W wavefronts through
// LDS.  Contains a barrier.  nm: the lane's negated minimum (taken before the columns past M were masked).
template <int W>
struct BoundsLds {
  float hi[W], nlo[W], nt0[W], probe[W];
};
template <int E, int W, bool NEG, bool FILTER, int J>
__device__ __forceinline__ void block_bounds(const float (&x)[E], float nm, int need, int lane, int wave, BoundsLds<W>& s,
                                             float& lo, float& hi, float& T0, float& probe) {
  float gm[J], wmax, wmin, above = 0.0f, floor_w = 0.0f;
  lane_group_maxima<E, NEG>(x, gm);
  float mx = gm[0];
#pragma unroll
  for (int j = 1; j < J; ++j) mx = vmax(mx, gm[j]);
  wave_max_and_negmin(mx, nm, wmax, wmin);
  if constexpr (FILTER) floor_w = floor_of_maxima<J>(gm, need, wmin, wmax, above);
  if (lane == 0) {
    s.hi[wave] = wmax;
    s.nlo[wave] = -wmin;
    if constexpr (FILTER) {
      s.nt0[wave] = -floor_w;
      s.probe[wave] = above;
    }
  }
  __syncthreads();
  float a = s.hi[0], b = s.nlo[0], c = 0.0f, d = 0.0f;
#pragma unroll
  for (int w = 1; w < W; ++w) {
    a = vmax(a, s.hi[w]);
    b = vmax(b, s.nlo[w]);
  }
  if constexpr (FILTER) {
    c = s.nt0[0], d = s.probe[0];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      c = vmax(c, s.nt0[w]);
      d = vmax(d, s.probe[w]);
    }
  }
  // every lane holds the same values; saying so lets the search loops branch on scalar conditions
  hi = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a)));
  lo = -__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(b)));
  T0 = -__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(c)));
  probe = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(d)));
}

// What is known of a search before a row's full-width pass: where Algorithm 2, or Algorithm 1 with precision, has ended.
struct KnownBounds {
  int known;  // 0: nothing
  float lo, hi;
  int iterations;
};

// One row, by the whole workgroup; true when it is done (always, but for kListsOnly, which leaves in `bounds` what it knows; the
// full-width search leaves the selection's lowest threshold in bounds.lo).  Every wavefront leaves through the
// same return statement.  A workgroup that walks several rows through the lists loads the whole next row as soon as the
// list of quads stands, into the registers of this one (have_next: x holds the row on entry); with the full-width
// search, as much of the next row as fits beside this one is loaded while this one is ranked (ahead).  shares: floor_shares(); with
// kListsOnly the wavefront's own share.
template <int G, int NG, int W, int MODE, bool NEG, int DT, bool DENSE, int PATH, int ROOM = list_room(W)>
__device__ __forceinline__ bool block_row(int64_t r, const void* __restrict__ in, int64_t N, int M, int k, int max_iter,
                                          float eps_rel, void* __restrict__ out_vals, int32_t* __restrict__ out_idx,
                                          int32_t* __restrict__ out_iters, uint32_t shares, int64_t r_next, bool& have_ahead,
                                          float (&ahead)[block_groups_ahead(W, G, PATH) * G + 1], bool& have_next,
                                          float (&x)[G * NG], KnownBounds& bounds) {
  static_assert(!DENSE || DT == kF32, "the dense form is built for fp32 rows");
  constexpr int E = G * NG;
  constexpr bool FILTER = PATH != kFullWidth;
  constexpr int T = NG * W;  // (group, wavefront) cells of a row, in column order
  constexpr int CPL = (T + kWave - 1) / kWave;  // cells per lane when one wavefront scans the table
  using ElemT = typename std::conditional<DT == kF32, float, uint16_t>::type;
  __shared__ BoundsLds<W> s_bounds;
  __shared__ typename std::conditional<FILTER, FilterLds<W, ROOM>, int>::type s_filter;
  __shared__ int s_cnt[2][W];          // per-wavefront counts of a search step, double buffered
  __shared__ int s_tab[2][T];          // candidates per cell of class A / class B, then their exclusive prefixes
  // narrowing of Algorithm 1's search (see gather_band): the whole row's band, its size, and what
  // wavefront 0 hands back after finishing the search alone
  __shared__ float s_band[kBandRegs * kWave + W * kWave];  // the row's band, then one dummy word per lane of the workgroup
  __shared__ int s_tot[2];  // band members / elements at or above hi, summed over the wavefronts
  __shared__ float s_res[3];
  __shared__ int s_resi[2];

  int lane = threadIdx.x & (kWave - 1);
  asm volatile("" : "+v"(lane));  // opaque per row: nothing derived from it is carried around the loop over rows
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const ElemT* row = static_cast<const ElemT*>(in) + r * (int64_t)M;

  // Loading stage.  The row, or its first groups, may have been loaded already, while the workgroup's previous row
  // was ranked.
  constexpr int AHEAD = block_groups_ahead(W, G, PATH) < NG ? block_groups_ahead(W, G, PATH) : NG;
  if (!FILTER || !have_next) {  // uniform
    if (AHEAD > 0 && have_ahead) {
#pragma unroll
      for (int e = 0; e < AHEAD * G; ++e) x[e] = ahead[e];
    } else {
      block_load<DT, G, W, 0, AHEAD>(row, M, lane, wave, x);
    }
    block_load<DT, G, W, AHEAD, NG>(row, M, lane, wave, x);
  }
  have_next = false;
  int need = 0;
  if constexpr (PATH == kListsFirst) {
    need = floor_share(M, G, W, wave, shares);
    asm volatile("" : "+s"(need));  // here, while the loads are in flight (after them it costs 0.1 us)
  } else if constexpr (PATH == kListsOnly) {
    need = (int)shares;
  }

  const float nm = lane_negmin<E, NEG>(x);
  block_mask<G, NG, W, NEG>(x, M, lane, wave);
  if (threadIdx.x == 0) {
    s_tot[0] = 0;
    s_tot[1] = 0;
    if constexpr (FILTER) {
      s_filter.n_quads = 0;
      s_filter.n_singles = 0;
    }
  }
  float hi, lo, T0, probe;
  constexpr int J = floor_groups(E, ROOM > list_room(W));
  block_bounds<E, W, NEG, FILTER, J>(x, nm, need, lane, wave, s_bounds, lo, hi, T0, probe);
  const float least = lo;

  using OutT = typename std::conditional<DT == kF32, uint32_t, uint16_t>::type;  // value bits as stored
  OutT* ov = static_cast<OutT*>(out_vals) + r * (int64_t)(DENSE ? M : k);
  int32_t* oi = DENSE ? nullptr : out_idx + r * (int64_t)k;
  have_ahead = false;
  auto next_ahead = [&]() {  // the first groups of the workgroup's next row
    if constexpr (AHEAD > 0) {
      if (r_next < N) {
        block_load<DT, G, W, 0, AHEAD>(static_cast<const ElemT*>(in) + r_next * (int64_t)M, M, lane, wave, ahead);
        have_ahead = true;
      }
    }
  };
  if constexpr (FILTER) {
    float thi, tlo;
    int split, iterations = 0;
    const float eps = MODE == kEps ? eps_rel * __builtin_fabsf(hi) : 0.0f;
    auto column = [&](int quad, int thread) -> int {
      const int g = quad / (G / 4);
      return min((g * W * kWave + thread) * G, M - G) + 4 * (quad % (G / 4));
    };
    // once the list of quads stands, the whole next row is loaded while this one is searched and written
    auto listed = [&]() {
      if constexpr (PATH == kListsOnly && !DENSE) {
        if (r_next < N) {
          __builtin_amdgcn_sched_barrier(0);  // not before the list has this row's values
          block_load<DT, G, W, 0, NG>(static_cast<const ElemT*>(in) + r_next * (int64_t)M, M, lane, wave, x);
          have_next = true;
        }
      }
    };
    auto emit = [&](int place, uint32_t value, int col) {
      if constexpr (DT == kF32) {
        ov[place] = value;
      } else {
        ov[place] = (uint16_t)narrow_bits<DT>(value);
      }
      oi[place] = col;
    };
    const int done = filter_row<E, W, ROOM, MODE, NEG, DT, DENSE>(s_filter, x, lane, wave, k, max_iter, eps, T0, probe, lo, hi,
                                                            thi, tlo, split, iterations, column, listed, emit);
    if (done == kFilterDone) {
      if constexpr (MODE == kEps) {
        if (out_iters != nullptr && threadIdx.x == 0) out_iters[r] = iterations;
      }
      if constexpr (DENSE) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          int ln = lane;  // opaque per group: keeps the column numbers of all groups from being hoisted
          asm volatile("" : "+v"(ln));
          const int col = ((g * W + wave) * kWave + ln) * G, col0 = min(col, M - G);
          float y[G];
#pragma unroll
          for (int c = 0; c < G; ++c) y[c] = x[g * G + c] >= (col0 + c <= split ? tlo : thi) ? x[g * G + c] : 0.0f;
          store_row_group<G>(reinterpret_cast<float*>(ov), col, M, y);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      return true;
    }
    bounds.known = MODE != kExact && done == kFilterBoundOnly ? 1 : 0;
    bounds.lo = lo;
    bounds.hi = hi;
    bounds.iterations = iterations;
    if constexpr (PATH == kListsOnly) return false;
  }
  if (MODE != kExact && bounds.known != 0) {
    lo = bounds.lo;
    hi = bounds.hi;
  }

  // cnt = #{row elements with key >= t}.  Every lane counts its keys below t, the wavefront sums them,
  // lane 0 posts the sum, and after the barrier every wavefront adds up the W posted sums itself (they sit
  // in one row of 16 lanes).  `step` selects the half of s_cnt that is written; one barrier per step is
  // enough because a half is not written again before every wavefront has passed the next barrier.
  // (Adding the lanes' counts to one LDS word with atomics instead, which saves the second reduction,
  // measured slower: 8192 x 32768 at eight steps 252 -> 266 us.)
  int step = 0;
  constexpr int kPackWords = (E + 31) / 32;
  uint32_t last[kPackWords];  // this lane's sign-bit words of the latest count
  auto count = [&](float t) -> int {
    lane_below_packs<E, NEG>(x, t, last);
    uint32_t below_lane = 0;
#pragma unroll
    for (int g = 0; g < kPackWords; ++g) below_lane += (uint32_t)__builtin_popcount(last[g]);
    const int mine = wave_sum((int)below_lane);
    const int p = step & 1;
    ++step;
    if (lane == 0) s_cnt[p][wave] = mine;
    __syncthreads();
    const int below = __builtin_amdgcn_readfirstlane((int)row16_sum(lane < W ? (uint32_t)s_cnt[p][lane] : 0u));
    return W * kWave * E - below;  // padded columns hold a key of -inf and are among the `below`
  };

  // The selection is described by two classes of elements and a limit for each:
  //   class A: key >= tA, the first limA of them in column order are chosen;
  //   class B: tB <= key < tA, the first limB of them are chosen (only after a converged search).
  float tA, tB = 0.0f;
  int limA = k, limB = 0;
  if constexpr (MODE == kExact || MODE == kEps) {
    // Algorithm 1; termination, collection and iteration numbering as in select_row.  The full-width
    // steps track cnt_lo = #{key >= lo} and a lower bound cnt_hi of #{key >= hi}; once the band
    // [lo, hi) of the whole row fits kBandRegs registers per lane of ONE wavefront, it is gathered
    // there and wavefront 0 finishes the search alone, with no further barriers.
    bool hit = false, narrow = false;
    float thres = lo;
    int steps = MODE == kEps && bounds.known != 0 ? bounds.iterations - 1 : 0, cnt_lo = M, cnt_hi = 0;
    const float eps = MODE == kEps ? eps_rel * __builtin_fabsf(hi) : 0.0f;
    // (Narrowing as soon as the band fits stays the fastest: never narrowing costs 3 % on Laplace rows --
    // 12.3 full-width steps on average at 32768 columns -- and starting only after 8 to 14 steps 7-12 %.
    // Narrowing three to four steps earlier, onto kBandRegs registers per lane of EVERY wavefront with the
    // remaining steps still going through the barrier, measured slower as well: 8192 x 32768 249 -> 263 us,
    // 4096 x 65536 319 -> 350 us; a step on one wavefront's registers costs a tenth of a step that all
    // wavefronts have to meet for.)
    // the sign-bit words of the steps that set the current lo and hi: the gather needs no compare of its own
    uint32_t below_lo[kPackWords], below_hi[kPackWords];
    bool lo_moved = false, hi_moved = false;
    auto fits = [&](int cnt) -> bool {  // after move_bound with this count
      if (cnt < k) {  // uniform
        hi_moved = true;
#pragma unroll
        for (int g = 0; g < kPackWords; ++g) below_hi[g] = last[g];
      } else {
        lo_moved = true;
#pragma unroll
        for (int g = 0; g < kPackWords; ++g) below_lo[g] = last[g];
      }
      cnt_lo = cnt < k ? cnt_lo : cnt;
      cnt_hi = cnt < k ? cnt : cnt_hi;
      return cnt_lo - cnt_hi <= kBandRegs * kWave;
    };
    if constexpr (MODE == kExact) {
      float seen = lo;
      for (;;) {
        thres = midpoint_exact<DT>(lo, hi);
        if (!(thres < seen || thres > seen)) break;
        seen = thres;
        int cnt = count(thres);
        if (cnt == k) {
          hit = true;
          break;
        }
        move_bound(lo, hi, thres, cnt, k);
        if (fits(cnt)) {
          narrow = true;
          break;
        }
        thres = midpoint_exact<DT>(lo, hi);
        cnt = count(thres);
        if (cnt == k) {
          hit = true;
          break;
        }
        move_bound(lo, hi, thres, cnt, k);
        if (fits(cnt)) {
          narrow = true;
          break;
        }
      }
    } else {
      while (bounds.known == 0 && hi - lo > eps) {
        const float mid = (lo + hi) * 0.5f;
        if (!(mid > lo && mid < hi)) break;
        thres = mid;
        ++steps;
        const int cnt = count(thres);
        if (cnt == k) {
          hit = true;
          break;
        }
        move_bound(lo, hi, thres, cnt, k);
        if (fits(cnt)) {
          narrow = true;
          break;
        }
      }
    }
    if (narrow) {  // uniform over the workgroup
      // every wavefront appends its band members to the row's band (any order will do)
      const uint32_t dst = (uint32_t)(uintptr_t)s_band;
      if (!lo_moved) lane_below_packs<E, NEG>(x, lo, below_lo);  // a bound still at the row's minimum or maximum
      if (!hi_moved) lane_below_packs<E, NEG>(x, hi, below_hi);
      scatter_band_members<E, NEG>(x, below_lo, below_hi, lane, dst + (uint32_t)((kBandRegs + wave) * kWave) * 4u,
                                   [&](uint32_t n, uint32_t above) -> uint32_t {
                                     uint32_t off = 0;
                                     if (lane == 0) {
                                       off = (uint32_t)atomicAdd(&s_tot[0], (int)n);
                                       atomicAdd(&s_tot[1], (int)above);
                                     }
                                     off = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
                                     return off + n <= (uint32_t)(kBandRegs * kWave) ? dst + off * 4u : kNoRoom;
                                   });
      __syncthreads();
      if (wave == 0) {
        float all[kBandRegs];
        const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane(s_tot[0]);
        const int above_all = __builtin_amdgcn_readfirstlane(s_tot[1]);
        load_band<NEG, kBandRegs>(dst, lane, total, all);
        search_band<MODE, NEG, DT, kBandRegs>(all, above_all, k, eps, lo, hi, thres, hit, steps);
        if (lane == 0) {
          s_res[0] = lo;
          s_res[1] = hi;
          s_res[2] = thres;
          s_resi[0] = hit ? 1 : 0;
          s_resi[1] = steps;
        }
      }
      __syncthreads();
      lo = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s_res[0])));
      hi = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s_res[1])));
      thres = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s_res[2])));
      hit = __builtin_amdgcn_readfirstlane(s_resi[0]) != 0;
      steps = __builtin_amdgcn_readfirstlane(s_resi[1]);
    }
    if constexpr (MODE == kEps) {
      if (out_iters != nullptr && threadIdx.x == 0) out_iters[r] = hit ? steps : steps + 1;
    }
    if (hit) {
      tA = thres;
    } else {
      const int na = count(hi);
      tA = hi;
      tB = not_below(lo, least);
      limA = na < k ? na : k;
      limB = k - limA;
    }
  } else {
    // Algorithm 2: max_iter steps (fewer once a step counts exactly k), then the first k of key >= lo.
    // (Counting the midpoint and both midpoints that can follow it in one pass -- two levels per barrier,
    // three counts per element -- gives the same bounds but measured slower, 250 -> 276 us at eight steps on
    // 8192 x 32768: a step is bound by its counting work, not by the barrier.)
#pragma nounroll
    for (int it = 0; bounds.known == 0 && it < max_iter; ++it) {
      const float thres = (lo + hi) * 0.5f;
      const int cnt = count(thres);
      move_bound(lo, hi, thres, cnt, k);
      if (cnt == k) break;
    }
    tA = not_below(lo, least);
  }
  if (PATH == kFullWidth) bounds.lo = limB > 0 ? tB : tA;
  // The search is over; what follows needs few registers besides the row.  A workgroup that has another
  // row to do starts that row's first loads now, so that they fly while this row is ranked and stored.
  next_ahead();
  const bool has_b = limB > 0;  // uniform over the workgroup

  // Ranking, part 1: candidates per (group, wavefront) cell, written in column order.
  //
  // One class (every search that ended on a count of k, and Algorithm 2): all per lane.  Each lane takes
  // its elements' candidate bits from the sign of key - tA, counts them per group, and the counts of up to
  // three groups share one word (10 bits each: a wavefront holds at most 64 * 8 candidates of a group)
  // through one prefix scan over the lanes.  The scan's last lane holds the cell totals, every lane keeps
  // the candidates in lower lanes for part 3.  Against one mask, one scalar popcount and one scalar add per
  // ELEMENT this leaves the scalar unit, which the 16 wavefronts of two rows share, nearly idle.
  constexpr int kScanWords = (NG + 2) / 3;
  uint32_t cand[(E + 31) / 32];          // candidate bits of this lane
  uint32_t lower[kScanWords];            // per group, 10 bits each: candidates of the cell in lower lanes
  uint32_t cell_total[kScanWords];       // the same fields for the whole wavefront (uniform)
  if (!has_b) {
    lane_bits_at_or_above<E, NEG>(x, tA, cand);
    uint32_t own[kScanWords];
#pragma unroll
    for (int j = 0; j < kScanWords; ++j) own[j] = 0;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      own[g / 3] |= (uint32_t)__builtin_popcount(group_bits<E, G>(cand, g)) << (10 * (g % 3));
#pragma unroll
    for (int j = 0; j < kScanWords; ++j) {
      const uint32_t incl = wave_inclusive_scan_dpp(own[j]);
      lower[j] = incl - own[j];  // field by field: no field borrows, incl >= own in each
      cell_total[j] = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (lane < NG) {
      // lane g posts cell g (the totals are uniform; the shift is per lane)
      uint32_t word = cell_total[0];
#pragma unroll
      for (int j = 1; j < kScanWords; ++j) word = lane / 3 == j ? cell_total[j] : word;
      s_tab[0][lane * W + wave] = (int)((word >> (10 * (lane % 3))) & 0x3ffu);
    }
  } else {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      int nA = 0, nB = 0;
#pragma unroll
      for (int c = 0; c < G; ++c) {
        const float v = keyof<NEG>(x[g * G + c]);
        nA += __builtin_popcountll(__builtin_amdgcn_ballot_w64(v >= tA));
        if (has_b) nB += __builtin_popcountll(__builtin_amdgcn_ballot_w64(v >= tB && !(v >= tA)));
      }
      if (lane == 0) {
        s_tab[0][g * W + wave] = nA;
        s_tab[1][g * W + wave] = nB;
      }
      if constexpr (NG > 4) __builtin_amdgcn_sched_barrier(0);  // keep the groups' masks from piling up
    }
  }
  __syncthreads();
  // Part 2: exclusive prefix over the cells (wavefront 0 scans class A, wavefront 1 class B).
  if (wave < 2) {
    int* tab = s_tab[wave];
    int v[CPL], sum = 0;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int f = lane * CPL + j;
      v[j] = f < T ? tab[f] : 0;
      sum += v[j];
    }
    int before = wave_inclusive_scan(sum, lane) - sum;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int f = lane * CPL + j;
      if (f < T) tab[f] = before;
      before += v[j];
    }
  }
  __syncthreads();

  // Part 3: every wavefront ranks its own elements.  Pairs go straight to the outputs at 4 (or 2) bytes
  // times their rank (k can be far larger than LDS could stage; consecutive ranks fall on consecutive
  // lanes, so the stores are still mostly coalesced); the dense form keeps or zeroes each element in
  // place and stores the row with the accesses it was loaded with.
  if (!has_b) {
    // One class, per lane: rank = cell prefix + candidates of the cell in lower lanes + own earlier
    // candidates in the group.  A lane's non-candidates get rank 0xffffffff, so that the one compare against
    // limA (which also keeps every store inside the row's k slots whatever the input held) decides who
    // stores.  Cells without a candidate are skipped as a whole.
    // (opaque copies: otherwise the group fields extracted in part 1 are kept in 16 registers for reuse here)
#pragma unroll
    for (int i = 0; i < (E + 31) / 32; ++i) asm volatile("" : "+v"(cand[i]));
    // lane g fetches the prefix of cell g: one LDS round trip for all the wavefront's cells
    const int my_cell = s_tab[0][(lane < NG ? lane : 0) * W + wave];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if constexpr (!DENSE) {
        if (((cell_total[g / 3] >> (10 * (g % 3))) & 0x3ffu) == 0) continue;  // uniform
      }
      int ln = lane;  // opaque per group: keeps the column numbers of all groups from being hoisted
      if constexpr (NG > 4) asm volatile("" : "+v"(ln));
      const uint32_t bits = group_bits<E, G>(cand, g);
      const uint32_t before = (uint32_t)__builtin_amdgcn_readlane(my_cell, g) +
                              __builtin_amdgcn_ubfe(lower[g / 3], (uint32_t)(10 * (g % 3)), 10u);
      const int col = ((g * W + wave) * kWave + ln) * G, col0 = min(col, M - G);
      float y[G];
      auto one = [&](auto cc) {
        constexpr int c = decltype(cc)::value;
        const uint32_t pos = before + (c == 0 ? 0u : (uint32_t)__builtin_popcount(bits >> (G - c)));
        const uint32_t is_cand = (uint32_t)__builtin_amdgcn_sbfe(bits, (uint32_t)(G - 1 - c), 1u);  // all ones or zero
        const uint32_t rank = pos | ~is_cand;
        if constexpr (DENSE) {
          y[c] = rank < (uint32_t)limA ? x[g * G + c] : 0.0f;
        } else {
          const uint32_t fb = __float_as_uint(x[g * G + c]);
          uint32_t vb = fb;
          if constexpr (DT != kF32) vb = narrow_bits<DT>(fb);
          store_pair_if_below<DT, c>(rank, (uint32_t)limA, ov, vb, oi, col0);
        }
      };
      static_for<G>(one);
      if constexpr (DENSE) store_row_group<G>(reinterpret_cast<float*>(ov), col, M, y);
      if constexpr (NG > 4) __builtin_amdgcn_sched_barrier(0);
    }
    return true;
  }
  // Two classes (a search that converged on a value tied across the k-th place): rare, kept plain.
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    uint32_t posA = (uint32_t)s_tab[0][g * W + wave];
    uint32_t posB = (uint32_t)s_tab[1][g * W + wave];
    bool a[G], b[G];
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const float v = keyof<NEG>(x[g * G + c]);
      a[c] = v >= tA;
      b[c] = v >= tB && !a[c];
      posA = lanes_below(__builtin_amdgcn_ballot_w64(a[c]), posA);
      posB = lanes_below(__builtin_amdgcn_ballot_w64(b[c]), posB);
    }
    const int col = ((g * W + wave) * kWave + lane) * G, col0 = min(col, M - G);
    float y[G];
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const uint32_t selA = posA < (uint32_t)limA ? posA : (uint32_t)limA;  // chosen A's before this element
      const uint32_t selB = posB < (uint32_t)limB ? posB : (uint32_t)limB;
      const bool chosen = (a[c] && posA < (uint32_t)limA) || (b[c] && posB < (uint32_t)limB);
      if constexpr (DENSE) {
        y[c] = chosen ? x[g * G + c] : 0.0f;
      } else {
        if (chosen) {
          const uint32_t pos = selA + selB;
          const uint32_t fb = __float_as_uint(x[g * G + c]);
          uint32_t bits = fb;
          if constexpr (DT != kF32) bits = narrow_bits<DT>(fb);
          ov[pos] = (OutT)bits;
          oi[pos] = col0 + c;
        }
      }
      posA += a[c] ? 1u : 0u;
      posB += b[c] ? 1u : 0u;
    }
    if constexpr (DENSE) store_row_group<G>(reinterpret_cast<float*>(ov), col, M, y);
    if constexpr (NG > 4) __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

// Workgroup b takes rows b, b + gridDim.x, ...: with as many workgroups as rows each takes one; the widest
// shape (16 wavefronts, one workgroup to a compute unit) is launched with one workgroup per compute unit
// instead, which saves the dispatch of a new 1024-thread workgroup between a unit's rows.  There the rows that the lists
// do not hold wait until up to 64 have been through: they are read again then, so that the lists' loop needs registers
// for no more than one row at a time.
template <int G, int NG, int W, int MODE, bool NEG, int DT, bool DENSE, bool FILTER, int ROOM = list_room(W)>
__device__ __forceinline__ void block_rows(const void* __restrict__ in, int64_t N, int M, int k, int max_iter,
                                           float eps_rel, void* __restrict__ out_vals, int32_t* __restrict__ out_idx,
                                           int32_t* __restrict__ out_iters, uint32_t shares) {
  bool have_ahead = false, have_next = false;
  KnownBounds bounds{};
  if constexpr (block_persistent(W) && FILTER) {
    __shared__ KnownBounds s_known[64];
    int need = floor_share(M, G, W, __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), shares);
    asm volatile("" : "+s"(need));  // once for all rows
    float x[G * NG];
    for (int64_t r0 = blockIdx.x; r0 < N; r0 += 64 * (int64_t)gridDim.x) {
      uint64_t left = 0;  // uniform: rows for the full-width pass
      have_next = false;
      for (int j = 0; j < 64; ++j) {
        const int64_t r = r0 + j * (int64_t)gridDim.x;
        if (r >= N) break;
        float none[1];
        const bool done = block_row<G, NG, W, MODE, NEG, DT, DENSE, kListsOnly, ROOM>(
            r, in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters, (uint32_t)need, j + 1 < 64 ? r + gridDim.x : N, have_ahead, none,
            have_next, x, bounds);
        left |= done ? 0ull : 1ull << j;
        if (!done && threadIdx.x == 0) {
          s_known[j].known = bounds.known;
          s_known[j].lo = bounds.lo;
          s_known[j].hi = bounds.hi;
          s_known[j].iterations = bounds.iterations;
        }
        __syncthreads();  // the next row reuses the shared tables
      }
      while (left != 0) {
        const int j = __builtin_ctzll(left);
        left &= left - 1;
        float ahead[block_groups_ahead(W, G, kFullWidth) * G + 1];
        have_ahead = false;
        bounds.known = __builtin_amdgcn_readfirstlane(s_known[j].known);
        bounds.lo = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s_known[j].lo)));
        bounds.hi = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s_known[j].hi)));
        bounds.iterations = __builtin_amdgcn_readfirstlane(s_known[j].iterations);
        block_row<G, NG, W, MODE, NEG, DT, DENSE, kFullWidth>(r0 + j * (int64_t)gridDim.x, in, N, M, k, max_iter, eps_rel,
                                                              out_vals, out_idx, out_iters, 0, N, have_ahead, ahead, have_next, x,
                                                              bounds);
        __syncthreads();
      }
    }
  } else if constexpr (block_persistent(W)) {
    float ahead[block_groups_ahead(W, G, kFullWidth) * G + 1], x[G * NG];
    for (int64_t r = blockIdx.x; r < N; r += gridDim.x) {
      block_row<G, NG, W, MODE, NEG, DT, DENSE, kFullWidth>(r, in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters,
                                                            0, r + gridDim.x, have_ahead, ahead, have_next, x, bounds);
      __syncthreads();  // the next row reuses the shared tables
    }
  } else {
    float none[1], x[G * NG];
    const int64_t r = blockIdx.x;  // launched with one workgroup per row
    if (r < N)
      block_row<G, NG, W, MODE, NEG, DT, DENSE, FILTER ? kListsFirst : kFullWidth, ROOM>(
          r, in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters, shares, N, have_ahead, none, have_next, x, bounds);
  }
}

// The full-width search alone (k too large for the lists), and the same behind the lists.
template <int G, int NG, int W, int MODE, bool NEG, int DT, bool DENSE>
__global__ void __launch_bounds__(W * kWave) __attribute__((amdgpu_waves_per_eu(block_persistent(W) ? 4 : 1)))
    rtopk_block_kernel(const void* __restrict__ in, int64_t N, int M, int k, int max_iter, float eps_rel,
                       void* __restrict__ out_vals, int32_t* __restrict__ out_idx, int32_t* __restrict__ out_iters) {
  block_rows<G, NG, W, MODE, NEG, DT, DENSE, false>(in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters, 0);
}
template <int G, int NG, int W, int MODE, bool NEG, int DT, bool DENSE>
__global__ void __launch_bounds__(W * kWave) __attribute__((amdgpu_waves_per_eu(block_persistent(W) ? 4 : 5)))
    rtopk_filter_kernel(const void* __restrict__ in, int64_t N, int M, int k, int max_iter, float eps_rel,
                        void* __restrict__ out_vals, int32_t* __restrict__ out_idx, int32_t* __restrict__ out_iters,
                        uint32_t shares) {
  block_rows<G, NG, W, MODE, NEG, DT, DENSE, true>(in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters, shares);
}

// Longer lists, for larger k; floors from groups of eight values, more of them than k needs.
template <int G, int NG, int W, bool NEG, int DT, int MODE>
__global__ void __launch_bounds__(W * kWave) __attribute__((amdgpu_waves_per_eu(4)))
    rtopk_filter_big_kernel(const void* __restrict__ in, int64_t N, int M, int k, int max_iter, float eps_rel,
                            void* __restrict__ out_vals, int32_t* __restrict__ out_idx, int32_t* __restrict__ out_iters,
                            uint32_t shares) {
  block_rows<G, NG, W, MODE, NEG, DT, false, true, big_list_room(W)>(in, N, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters,
                                                                     shares);
}

// Compute units of the current device (asked once per device; concurrent first calls store the same value).
inline int compute_units() {
  static int units[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (units[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    units[dev] = n;
  }
  return units[dev];
}

#ifndef RTOPK_BLOCK_PERSIST
#define RTOPK_BLOCK_PERSIST 1
#endif
template <int G, int NG, int W, int MODE, bool NEG = false, int DT = kF32, bool DENSE = false>
hipError_t launch_block(const LaunchArgs& a) {
  if (a.N > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  int64_t grid = a.N;
  if (RTOPK_BLOCK_PERSIST && block_persistent(W)) {
    const int64_t resident = (int64_t)compute_units() * (16 / W);  // workgroups that run at the same time
    if (resident > 0 && grid > resident) grid = resident;
  }
  constexpr int K = block_kernels(G * NG, W, MODE, DENSE, DT != kF32);
  static_assert(block_persistent(W) == (W == 16), "block_search knows the shape that walks its rows by its wavefronts");
  Shape s{};
  s.g = G;
  s.ng = NG;
  s.w = W;
  const int search = block_search(s, a.M, a.k, DT, MODE, a.max_iter, DENSE, a.N, a.eps_rel);
  auto launch = [&](auto kernel, auto... shares) {
    return launch_kernel(kernel, dim3((unsigned)grid), dim3(W * kWave), 0, a.stream, a.in, a.N, a.M, a.k, a.max_iter, a.eps_rel,
                         a.out_vals, static_cast<int32_t*>(a.out_idx), a.out_iters, shares...);
  };
  if constexpr ((K & kSearchRow) != 0) {
    if (search == kSearchRow) return launch(&rtopk_block_kernel<G, NG, W, MODE, NEG, DT, DENSE>);
  }
  if constexpr ((K & kSearchLists) != 0) {
    if (search == kSearchLists) return launch(&rtopk_filter_kernel<G, NG, W, MODE, NEG, DT, DENSE>, floor_shares(a.M, a.k, G));
  }
  if constexpr ((K & kSearchLongLists) != 0) {
    if (search == kSearchLongLists) return launch(&rtopk_filter_big_kernel<G, NG, W, NEG, DT, MODE>, floor_shares(a.M, a.k, G));
  }
  return hipErrorInvalidValue;
}

}  // namespace rtopk
