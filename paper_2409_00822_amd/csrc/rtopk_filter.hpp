// Selection of a wide row from the few elements that can matter (gfx950).  Included by rtopk_kernel.hpp, inside
// namespace rtopk, behind the cross-lane helpers; used by rtopk_kernel.hpp, rtopk_block_kernel.hpp and
// rtopk_split_kernel.hpp.
//
// Algorithms 1 and 2 (RTop-K, arXiv 2409.00822, Section 3.1) look at a count only to compare it with k.  For any
// floor T0 with more than k keys at or above it, the count at a threshold t <= T0 is therefore known to exceed k,
// and the count at t > T0 needs only the keys at or above T0.  A floor close to the k-th key costs almost nothing:
// every lane's maximum over a group of 16 elements is one element of the row, so the (k + 1)-th largest of those
// maxima has at least k + 1 keys at or above it -- and, being one of every 16th element's best, only about
// 1.2 to 1.4 k in all.  Finding it takes a bisection over E / 16 registers instead of E.  Then:
//   1. the floor: every wavefront bisects its own group maxima for its share of the k + 1 (no barrier), the row's
//      floor is the smallest of the wavefronts' floors (one exchange, the one that the minimum and maximum need);
//   2. the quads (four consecutive elements) with a key at or above the floor go to a list in LDS, any order: a
//      lane's quads are the set bits of one word, the lanes' counts are scanned, and every quad is stored -- members
//      to the lane's next slot, the others to a dummy slot of the lane -- with no lane mask and no branch;
//   3. their elements at or above the floor go to a list of (value, column) singles;
//   4. one wavefront runs the search on the singles, 64 to a register, with no barrier;
//   5. the winners' places in column order come from a bitmap over the row's columns: prefix popcounts.
// Thresholds, branches, exit iteration and result are those of the search over the whole row.  What a list does not
// hold (a row whose values crowd, k too large for the lists) is left to the caller's full-width search; where a search ends
// below the floor its bounds are the caller's, who selects by them.
//
// What bounds it: a row's elements are touched twice (maxima, then quad maxima against the floor; 5 vector
// instructions per four elements in all, and 8 plus two LDS writes per quad to store it) where the search over the
// whole row takes two instructions per element and STEP, 6 to 9 steps of them, a gather and a ranking of every
// element.  Issue time per wavefront of 64 values per lane falls from about 6000 cycles to about 1200.

// max of the keys a, b, c; of the key k and the keys a, b; and the same of the negated keys
template <bool NEG>
__device__ __forceinline__ float key_max3(float a, float b, float c) {
  return NEG ? vmax3_nnn(a, b, c) : vmax3(a, b, c);
}
template <bool NEG>
__device__ __forceinline__ float key_max3_on(float m, float a, float b) {
  return NEG ? vmax3_ann(m, a, b) : vmax3(m, a, b);
}
template <bool NEG>
__device__ __forceinline__ float key_max_on(float m, float a) {
  return NEG ? vmax_an(m, a) : vmax(m, a);
}

// Largest of the lane's negated keys (-min).
template <int E, bool NEG>
__device__ __forceinline__ float lane_negmin(const float (&x)[E]) {
  float nm = key_max3<!NEG>(x[0], x[1], x[2]);
#pragma unroll
  for (int e = 3; e + 1 < E; e += 2) nm = key_max3_on<!NEG>(nm, x[e], x[e + 1]);
  return E % 2 == 0 ? key_max_on<!NEG>(nm, x[E - 1]) : nm;
}

// Group maxima: gm[j] = largest key of the j-th of the lane's J groups of consecutive elements (see floor_groups, wave_groups).
template <int E, bool NEG, int J>
__device__ __forceinline__ void lane_group_maxima(const float (&x)[E], float (&gm)[J]) {
  constexpr int S = E / J;
  static_assert(E % J == 0 && S % 4 == 0, "whole groups of whole quads only");
#pragma unroll
  for (int j = 0; j < J; ++j) {
    float m = key_max3<NEG>(x[S * j], x[S * j + 1], x[S * j + 2]);
#pragma unroll
    for (int c = 3; c + 1 < S; c += 2) m = key_max3_on<NEG>(m, x[S * j + c], x[S * j + c + 1]);
    gm[j] = key_max_on<NEG>(m, x[S * j + S - 1]);
  }
}

// A floor under at least `need` of the wavefront's group maxima, as close to the need-th as a few steps bring it, between
// `low` (no larger than any key of the wavefront's) and `high` (its largest key); `above` is left at the lowest bound
// tried with fewer than `need` maxima at or above it.  Halving the range of values gets there in five to seven steps on
// ordinary rows (normal, Laplace, uniform; up to ten on squared distances) but not where one entry, or a masked part of the
// row, lies far from the others: from -1e9 twelve steps end at -2.4e5, below every other key, and the row would not fit the
// lists.  So the steps after the tenth take one of the group maxima between the bounds instead, which needs no more of
// them than any other values would (five to nine, 20 at most in 60 rows each of eleven kinds).  Exact mode with one entry of -1e9 a
// row, twelve halvings -> this: 8192 x 4096, k = 64, 74 -> 28 us; 1048 x 32000 102 -> 31; 671 x 50000, k = 100, 398 -> 40.
// (After seven halvings already: 2048 x 50000 squared distances, k = 100, 86.6 -> 89.6; now 87.5.)
// With NaN or infinite keys any value may come out.
// halvings: 0, or, where low and high are Algorithm 2's own first bounds, its number of steps if that is small: if they all
// move `low` they are that search, which ends there, below any better floor.
constexpr int kFloorHalvings = 10;
template <int J>
__device__ __forceinline__ float floor_of_maxima(const float (&gm)[J], int need, float low, float high, float& above,
                                                 int halvings = 0) {
  // (of a few maxima two more than needed will do: the slowest of 16 wavefronts that look for 7 takes 7 steps instead of 10.5,
  // and one row in ten no pivots, for 3 % more candidates)
  const int enough = need + (need >> 3) + (need < 32 ? 3 : 1);
  const float largest = high, least = low;
  auto at_or_above = [&](float t) -> int {
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) cnt += __builtin_popcountll(__builtin_amdgcn_ballot_w64(gm[j] >= t));
    return cnt;
  };
#pragma unroll  // (rolled, the steps of rows of 16 to 32 values per lane cost up to a tenth of their time)
  for (int step = 0; step < kFloorHalvings; ++step) {
    const float mid = (low + high) * 0.5f;
    const int cnt = at_or_above(mid);
    const bool enough_above = cnt >= need;  // (selects and one branch: a branch for each side costs 3 % at 16 values per lane)
    low = enough_above ? mid : low;
    high = enough_above ? high : mid;
    if ((uint32_t)(cnt - need) <= (uint32_t)(enough - need)) {
      above = high;
      return low < least ? least : low;  // (the sum of two bounds near the type's lowest value is -inf, which padding reaches too)
    }
  }
  // (A floor that is itself one of the keys leaves no room below the k-th for a precision-bounded search to end in, so
  // from here on two more maxima than needed: 7168 columns, k = 8, precision 1e-4 37 -> 27.)
  const int wanted = need + 2 + (need >> 4), at_most = enough + 3 + (need >> 4);
  bool found = false;
  auto try_bound = [&](float t) {
    const int cnt = at_or_above(t);
    if (cnt >= wanted) {
      low = t;
      found = cnt <= at_most;
    } else {
      high = t;
    }
  };
  for (int step = kFloorHalvings; step < halvings && !found; ++step) try_bound((low + high) * 0.5f);
  if (halvings != 0 && high == largest) found = true;
  for (int step = 0; step < 24 && !found; ++step) {
    // a lane's largest below `high`, or (every other step) its smallest above `low`
    const float inf = __builtin_inff();
    uint64_t lanes;
    float pick;
    if ((step & 1) == 0) {
      pick = -inf;
#pragma unroll
      for (int j = 0; j < J; ++j) pick = vmax(pick, gm[j] < high ? gm[j] : -inf);
      lanes = __builtin_amdgcn_ballot_w64(pick > low);
    } else {
      float neg = -inf;
#pragma unroll
      for (int j = 0; j < J; ++j) neg = vmax_an(neg, gm[j] > low ? gm[j] : inf);
      pick = -neg;
      lanes = __builtin_amdgcn_ballot_w64(pick < high);
    }
    if (lanes == 0) break;
    const int turn = (step * 29) & 63;  // the first of them from another lane on each time
    const uint64_t turned = (lanes >> turn) | (lanes << ((64 - turn) & 63));
    try_bound(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(pick), (__builtin_ctzll(turned) + turn) & 63)));
  }
  above = high;
  return low < least ? least : low;
}

// The steps of Algorithm 2, or of Algorithm 1 with precision eps, whose thresholds lie at or below the floor T0: each
// of them counts more than k keys and moves lo up.  Returns whether the search ends among them; then lo is final and hi
// still the largest key.  They are taken only if they may well be all there are -- if all steps but the last, halving [lo, hi] towards
// hi, or a last minimum within eps of hi, come out no higher than the floor: otherwise none is taken, and false returned,
// because the search on the lists takes them just as fast (16 values per lane, bfloat16, eight steps: 5 %).
template <int MODE>
__device__ __forceinline__ bool walk_to_floor(float T0, int max_iter, float eps, float& lo, float hi, int& steps) {
  steps = 0;
  const float reached = MODE == kEarly ? hi - __builtin_ldexpf(hi - lo, 1 - max_iter) : hi - eps;
  if (reached > T0) return false;
  for (;;) {
    if (MODE == kEarly ? steps >= max_iter : !(hi - lo > eps)) return true;
    const float mid = (lo + hi) * 0.5f;
    if (MODE == kEps && !(mid > lo && mid < hi)) return true;
    if (!(mid <= T0)) return false;
    lo = mid;
    ++steps;
  }
}

// The largest value on the row type's grid (see midpoint_exact) that is not above t.
template <int DT>
__device__ __forceinline__ float grid_floor(float t) {
  if constexpr (DT == kF32) {
    return t;
  } else {
    constexpr uint32_t mask = DT == kBF16 ? 0xffff0000u : 0xffffe000u;
    const uint32_t u = __float_as_uint(t), m = u & mask;
    return __uint_as_float(u != m && (u >> 31) != 0 ? m + ~mask + 1u : m);
  }
}

// ---- the k-th of a list by bins ---------------------------------------------------------------------------
//
// Exact mode does not depend on the thresholds, so its search on a list needs none: the keys are counted into 256 equal parts of
// [floor, largest key], one prefix sum over the parts finds the one with the k-th key, and the few members of that part are
// ranked against each other, ties by column.  That replaces 9 to 14 dependent steps of a compare, a popcount and an add per
// register.  The part of a key is a monotonic function of it, so rounding moves no key past another.  On the lists of a
// workgroup or a wavefront: 256 x 16384, k = 64 9.4 -> 8.2 us, bfloat16 8.1 -> 7.5; 256 x 32000, k = 64 12.0 -> 11.1; 2097 x 32000
// 48.4 -> 47.2, bfloat16 40.2 -> 37.9; 256 x 4096 6.8 -> 6.3, but 65536 x 4096, bound by its loads, 187 -> 186.  (16-bit rows of
// one wavefront search by steps: few values, so few steps and many members of a bin; 4096 columns 28.4 -> 28.9 with bins.  Of 16 values
// per lane likewise for k up to 8, whose lists fill one or two registers: 86037 x 780, k = 1 54.6 with bins, 50.5 by steps, k = 8 59.5
// and 55.6, k = 16 57 .. 59 either way; 2048 columns, 1000 rows, k = 8 5.8 and 6.1; not the dense form, 381 x 959, k = 7 5.3 and 5.5.)
constexpr int kBins = 256;  // part 0 holds the largest keys
__device__ __forceinline__ void clear_bins(uint32_t* count, int lane) {  // (16-byte aligned)
  reinterpret_cast<uint4*>(count)[lane] = make_uint4(0u, 0u, 0u, 0u);
}
__device__ __forceinline__ float bins_scale(float low, float high) { return (float)kBins * __builtin_amdgcn_rcpf(high - low); }
// (A NaN or a negative product converts to 0, one too large saturates.)
__device__ __forceinline__ int bin_of(float key, float high, float scale) {
  uint32_t b;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(b) : "v"((high - key) * scale));
  return (int)min(b, (uint32_t)kBins - 1u);
}
// The part that holds the k-th largest of the counted keys, -1 if there is none; `above`: keys in higher parts, in_bin: keys
// in it.  Called by whole wavefronts, behind a barrier (for one wavefront a fence).
__device__ __forceinline__ int find_bin(const uint32_t* count, int lane, int k, int& above, int& in_bin) {
  const uint4 c = reinterpret_cast<const uint4*>(count)[lane];
  const uint32_t a1 = c.x, a2 = a1 + c.y, a3 = a2 + c.z, sum = a3 + c.w;
  const uint32_t incl = wave_inclusive_scan_dpp(sum), before = incl - sum;
  const uint64_t owner = __builtin_amdgcn_ballot_w64(before < (uint32_t)k && (uint32_t)k <= incl);
  if (owner == 0) return -1;
  const int l = __builtin_ctzll(owner);
  const uint32_t want = (uint32_t)k - before;  // 1 .. sum in the owner
  const uint32_t part = (want > a1 ? 1u : 0u) + (want > a2 ? 1u : 0u) + (want > a3 ? 1u : 0u);
  const uint32_t first = want > a3 ? a3 : (want > a2 ? a2 : (want > a1 ? a1 : 0u));
  const uint32_t held = want > a3 ? c.w : (want > a2 ? c.z : (want > a1 ? c.y : c.x));
  above = __builtin_amdgcn_readlane((int)(before + first), l);
  in_bin = __builtin_amdgcn_readlane((int)held, l);
  return 4 * l + __builtin_amdgcn_readlane((int)part, l);
}
// The want-th (1-based) of the n members (key bits, column), at most 64 in any order, by key, then column: its key t and its
// column; cut: members equal to t rank behind it; NEXT: the key of the one that ranks next, if there is one.  Returns false
// where there is no such member (NaN keys).
template <bool NEXT = false>
__device__ __forceinline__ bool rank_members(const uint2* member, int lane, int n, int want, float& t, int& column, bool& cut,
                                             float& next) {
  const uint2 e = member[lane < n ? lane : 0];
  const float key = __uint_as_float(e.x);
  int rank = lane < n ? 0 : 2 * kWave;
  for (int q = 0; q < n; ++q) {
    const float other = __int_as_float(__builtin_amdgcn_readlane((int)e.x, q));
    const int other_col = __builtin_amdgcn_readlane((int)e.y, q);
    rank += (other > key || (other == key && other_col < (int)e.y)) ? 1 : 0;
  }
  const uint64_t at = __builtin_amdgcn_ballot_w64(rank == want - 1);
  if (at == 0) return false;
  const int l = __builtin_ctzll(at);
  t = __int_as_float(__builtin_amdgcn_readlane((int)e.x, l));
  column = __builtin_amdgcn_readlane((int)e.y, l);
  cut = __builtin_amdgcn_ballot_w64(lane < n && key == t && rank >= want) != 0;
  if constexpr (NEXT) {
    const uint64_t behind = __builtin_amdgcn_ballot_w64(rank == want);
    if (behind == 0) return want == n;
    next = __int_as_float(__builtin_amdgcn_readlane((int)e.x, __builtin_ctzll(behind)));
  }
  return true;
}

// The steps of Algorithm 2, or of Algorithm 1 with precision eps, from the k-th and the (k + 1)-th largest key alone: a
// threshold counts fewer than k keys where it lies above the k-th and more than k where it does not lie above the next, so no
// step has anything to count.  A step is half a dozen dependent instructions instead of a compare, a popcount and an add for each register
// of candidates, and in a workgroup a barrier.  steps: taken already, and then in all; hit: the last one, at thres, counted k.
template <int MODE>
__device__ __forceinline__ void steps_by_rank(float kth, float next, int max_iter, float eps, float& lo, float& hi,
                                              float& thres, bool& hit, int& steps) {
  hit = false;
  for (;;) {
    if (MODE == kEarly ? steps >= max_iter : !(hi - lo > eps)) break;
    const float mid = (lo + hi) * 0.5f;
    if (!(mid > lo && mid < hi)) {
      // no fp32 value strictly inside (lo, hi): Algorithm 1 ends; Algorithm 2's steps repeat one midpoint, equal to lo
      // (nothing moves) or to hi (lo moves up to it where hi itself counts k or more)
      if (MODE == kEarly && mid == hi && hi > lo && kth >= hi) lo = hi;
      break;
    }
    ++steps;
    if (mid > kth) {
      hi = mid;
    } else {
      thres = lo = mid;
      if (mid > next) {
        hit = true;
        break;
      }
    }
  }
}

// The smallest float above t (of a zero of either sign: the smallest above zero).
__device__ __forceinline__ float next_above(float t) {
  const int u = __float_as_int(t);
  return t == 0.0f ? __int_as_float(1) : __int_as_float(u < 0 ? u - 1 : u + 1);
}
// One wavefront: the k-th of the n singles (value bits, column), all at or above T0, hi the largest key.  bins: kBins words of
// LDS of its own, 16-byte aligned.  The selection is key >= (column <= split ? tlo : thi), or, with a limit above 0, key >= thi
// and the first `limit` of [tlo, thi) in column order (more than 64 equal keys; LEVELS = 3 only).  Returns false where it is
// not found: more than 64 members of its (last level's) bin, NaN keys.  (The singles are read twice rather than kept: the row
// is still in registers here, for the search that follows where this one fails.  BATCH: registers of them that are read
// together; LEVELS: of parts of parts.)
template <int BATCH, int LEVELS, bool NEG>
__device__ __forceinline__ bool kth_by_bins(const uint2* single, int n, int lane, int k, float T0, float hi, uint32_t* bins,
                                            float& thi, float& tlo, int& split, int& limit) {
  // Values with a heavy tail crowd in the last parts: a part with more members than can be ranked is cut into 256 again.
  limit = 0;
  static_assert(LEVELS == 1 || LEVELS == 3, "one level, or three");
  float top[3], scale[3];
  int chosen[3];
  top[0] = hi;
  scale[0] = bins_scale(T0, hi);
  int level = 0, above = 0, in_bin = 0;
  auto inside = [&](float key) -> bool {  // the parts chosen so far
    bool in = true;
#pragma unroll
    for (int l = 0; l + 1 < LEVELS; ++l)
      if (l < level) in = in && bin_of(key, top[l], scale[l]) == chosen[l];
    return in;
  };
  for (;;) {
    clear_bins(bins, lane);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i0 = 0; i0 < n; i0 += BATCH * kWave) {
      float key[BATCH];
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        const int j = i0 + i * kWave + lane;
        key[i] = keyof<NEG>(__uint_as_float(single[j < n ? j : 0].x));
      }
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        const int bin = bin_of(key[i], level == 0 ? top[0] : (level == 1 ? top[1] : top[2]),
                               level == 0 ? scale[0] : (level == 1 ? scale[1] : scale[2]));
        if (i0 + i * kWave + lane < n && (level == 0 || inside(key[i])))
          __hip_atomic_fetch_add(bins + bin, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int higher;
    const int part = find_bin(bins, lane, k - above, higher, in_bin);
    if (part < 0) return false;  // uniform
    above += higher;
    if (level == 0) chosen[0] = part;
    if (level == 1) chosen[1] = part;
    if (level == 2) chosen[2] = part;
    if (in_bin <= kWave) break;
    if (level + 1 == LEVELS) return false;
    // the members' own range is the next level's; are they all one value, the first of them in column order are chosen
    float largest = -__builtin_inff(), neg = -__builtin_inff();
    ++level;
    for (int i = lane; i < n; i += kWave) {
      const float key = keyof<NEG>(__uint_as_float(single[i].x));
      if (inside(key)) {
        largest = vmax(largest, key);
        neg = vmax_an(neg, key);
      }
    }
    --level;
    float t, least;
    wave_max_and_negmin(largest, neg, t, least);
    if (t == least) {
      tlo = t;
      thi = next_above(t);
      split = 0x7fffffff;
      limit = k - above;
      return true;
    }
    const float w = bins_scale(least, t);
    if (level == 0) {
      top[1] = t;
      scale[1] = w;
    } else {
      top[2] = t;
      scale[2] = w;
    }
    ++level;
  }
  ++level;  // all of them from here on
  uint2* member = reinterpret_cast<uint2*>(bins);
  uint32_t members = 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  for (int i0 = 0; i0 < n && members < (uint32_t)in_bin; i0 += BATCH * kWave) {
    uint2 e[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int j = i0 + i * kWave + lane;
      e[i] = single[j < n ? j : 0];
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float key = keyof<NEG>(__uint_as_float(e[i].x));
      const bool in = level == 1 ? bin_of(key, top[0], scale[0]) == chosen[0]
                                 : inside(key) && (level == 2 || bin_of(key, top[2], scale[2]) == chosen[2]);
      const uint64_t m = __builtin_amdgcn_ballot_w64(i0 + i * kWave + lane < n && in);
      if (m != 0) {  // uniform
        const uint32_t at = lanes_below(m, members);
        if (((m >> lane) & 1) != 0 && at < (uint32_t)kWave) member[at] = make_uint2(__float_as_uint(key), e[i].y);
        members += (uint32_t)__builtin_popcountll(m);
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  bool cut;
  float unused;
  if (!rank_members(member, lane, in_bin, k - above, tlo, split, cut, unused)) return false;
  thi = cut ? next_above(tlo) : tlo;
  if (!cut) split = 0x7fffffff;
  return true;
}

// #{singles with a key at or above t}, and the largest key below t (-inf if there is none), by one wavefront.
template <bool NEG>
__device__ __forceinline__ int count_singles(const uint2* single, int n, int lane, float t, float& below) {
  float neg = __builtin_inff(), largest = -__builtin_inff();
  int count = 0;
  for (int i0 = 0; i0 < n; i0 += 4 * kWave) {
    float key[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = i0 + i * kWave + lane;
      key[i] = keyof<NEG>(__uint_as_float(single[j < n ? j : 0].x));
      if (j >= n) key[i] = -__builtin_inff();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      count += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >= t));
      largest = key[i] < t ? vmax(largest, key[i]) : largest;
    }
  }
  wave_max_and_negmin(largest, neg, below, neg);
  return count;
}

// LDS of one row.  CAP: quads, and singles, that the lists hold (list_room, big_list_room).  The bitmaps take the quads' place when those
// have become singles.
template <int W, int ROOM = list_room(W)>
struct FilterLds {
  static constexpr int CAP = ROOM;
  static constexpr int WORDS = 128 * W;  // bitmap words: two per thread, 64 * 64 * W columns
  struct Lists {
    float4 quad[CAP + kWave];    // behind the list: a dummy slot per lane, shared by the wavefronts, never read
    uint32_t id[CAP + kWave];    // (quad of the lane) << 16 | thread
  };
  struct Maps {
    uint2 cut[WORDS / 2], chosen[WORDS / 2];
    uint32_t before[WORDS / 2];  // per thread: set bits in lower threads of its wavefront, and those plus its first word's
  };
  union {
    Lists lists;
    Maps maps;
  };
  uint2 single[CAP];             // (value bits, column)
  alignas(16) uint32_t bins[kBins];
  int n_quads, n_singles;
  int wave_bits[W];
  float thr[2];
  int info[3];                   // limit of the cut class (0: none), exit iteration, split column
  int state;
};

enum FilterResult : int {
  kFilterDone = 0,      // the pairs are written (or, in the dense form, the thresholds and the split are set)
  kFilterNoList = 1,    // the lists do not hold the row: the whole search is the caller's
  kFilterBoundOnly = 2  // the search is over without a count of k, but its last minimum lies below the floor: the selection is
                        // the caller's, from lo and hi (Algorithm 2: from lo)
};

// (filter_max_k of rtopk_shape.hpp: the largest k for the lists.  The floor has 1.4 to 1.6 k candidates at such k -- 1.2 to
// 1.35 k, and the spread of the wavefronts' floors; 2 k at k = 64: normal rows of 21848 columns in 8 wavefronts, k = 512: 824
// on average, 1012 at most in 200.)

// Positions of the set bits of one bitmap: `before` and `wave_bits` for the words of `map`.  Called by the whole
// workgroup with a barrier before it; contains one.
template <int W, int ROOM>
__device__ __forceinline__ void filter_prefix(FilterLds<W, ROOM>& s, const uint2* map, int lane, int wave) {
  const int tid = wave * kWave + lane;
  const uint2 w = map[tid];
  const uint32_t n0 = (uint32_t)__builtin_popcount(w.x), n = n0 + (uint32_t)__builtin_popcount(w.y);
  const uint32_t incl = wave_inclusive_scan_dpp(n);
  s.maps.before[tid] = (incl - n) | ((incl - n + n0) << 16);
  if (lane == kWave - 1) s.wave_bits[wave] = (int)incl;
  __syncthreads();
}
// Set bits of the map below column `col`.
template <int W, int ROOM>
__device__ __forceinline__ uint32_t filter_rank(const FilterLds<W, ROOM>& s, const uint2* map, int col) {
  const int word = col >> 5, owner = word >> 1;
  const uint32_t b = s.maps.before[owner];
  const uint2 w = map[owner];
  const uint32_t bits = (word & 1) ? w.y : w.x;
  uint32_t r = ((word & 1) ? b >> 16 : b & 0xffffu) + (uint32_t)__builtin_popcount(bits & ((1u << (col & 31)) - 1u));
  const int owner_wave = owner >> 6;
#pragma unroll
  for (int w2 = 0; w2 + 1 < W; ++w2) r += w2 < owner_wave ? (uint32_t)s.wave_bits[w2] : 0u;
  return r;
}

// Step 4, by one wavefront: the search on the singles.  SR registers per lane hold them; `steps` steps are done already.
template <int SR, int MODE, bool NEG, int DT>
__device__ __forceinline__ void filter_search(const uint2* single, int n, int lane, int k, int max_iter, float eps,
                                              float T0, float probe, float& lo, float& hi, float& thres, bool& hit,
                                              int& steps, int& last_cnt, int& na) {
  float key[SR];
#pragma unroll
  for (int i = 0; i < SR; ++i) {
    const int j = i * kWave + lane;
    const uint32_t v = single[j < n ? j : 0].x;
    key[i] = j < n ? keyof<NEG>(__uint_as_float(v)) : -__builtin_inff();
  }
  auto count = [&](float t) -> int {
    int c = 0;
#pragma unroll
    for (int i = 0; i < SR; ++i) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >= t));
    return c;
  };
  hit = false;
  last_cnt = -1;
  if constexpr (MODE == kEarly) {
    for (int it = steps; it < max_iter; ++it) {
      const float mid = (lo + hi) * 0.5f;
      const int cnt = mid > T0 ? count(mid) : k + 1;  // more than k keys are at or above the floor
      last_cnt = cnt;
      move_bound(lo, hi, mid, cnt, k);
      if (cnt == k) break;
    }
  } else {
    if constexpr (MODE == kExact) {
      // the answer does not depend on the thresholds: start at the floor, and try first the lowest bound that had
      // too few group maxima above it, which is usually just above the k-th key
      lo = grid_floor<DT>(T0);
      const float p = grid_floor<DT>(probe);
      if (p > lo && p < hi) {
        const int cnt = count(p);
        thres = p;
        if (cnt == k) hit = true;
        move_bound(lo, hi, p, cnt, k);
      }
    }
    while (!hit) {
      if constexpr (MODE == kEps) {
        if (!(hi - lo > eps)) break;
      }
      const float mid = MODE == kEps ? (lo + hi) * 0.5f : midpoint_exact<DT>(lo, hi);
      if (!(mid > lo && mid < hi)) break;
      thres = mid;
      ++steps;
      const int cnt = mid > T0 ? count(mid) : k + 1;
      if (cnt == k) hit = true;
      if (!hit) move_bound(lo, hi, mid, cnt, k);
    }
    na = hit ? k : count(hi);  // hi is at or above the floor: it is the largest key or has counted fewer than k
  }
}

// Steps 2 and 3 for one row, by the whole workgroup (W wavefronts): returns how many singles there are, -1 where a
// list does not hold them.  x: the row's elements, masked (a key of -inf past the row's end).  Before the call n_quads
// and n_singles are zero and a barrier has passed; the lists are complete for every wavefront on return.
// column(quad of the lane, thread): the quad's first column.  listed(): called once x is no longer needed here.  store =
// false: listed() is called, the lists are not built (-1).
template <int E, int W, bool NEG, int ROOM, typename Column, typename Listed>
__device__ __forceinline__ int filter_lists(FilterLds<W, ROOM>& s, const float (&x)[E], int lane, int wave, float T0,
                                            Column column, Listed listed, bool store = true) {
  constexpr int CAP = ROOM, Q = E / 4;
  static_assert(Q <= 32, "a lane's quads are the bits of one word");
  const int tid = wave * kWave + lane;

  // Step 2.  Bit Q - 1 - q of `member`: quad q has a key at or above T0 (the sign of key - T0, see count_ge_wide).
  {
    const float tz = T0 == 0.0f ? -0.0f : T0;
    uint32_t below = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float m = key_max_on<NEG>(key_max3<NEG>(x[4 * q], x[4 * q + 1], x[4 * q + 2]), x[4 * q + 3]);
      below = __builtin_amdgcn_alignbit(below, __float_as_uint(m - tz), 31);
    }
    uint32_t member = ~below & (Q == 32 ? 0xffffffffu : (1u << Q) - 1u);
    const uint32_t n_lane = (uint32_t)__builtin_popcount(member);
    const uint32_t incl = wave_inclusive_scan_dpp(n_lane);
    const int n_wave = __builtin_amdgcn_readlane((int)incl, kWave - 1);
    int base = 0;
    if (lane == 0) base = atomicAdd(&s.n_quads, n_wave);
    base = __builtin_amdgcn_readfirstlane(base);
    if (base + n_wave > CAP) member = 0;  // uniform: n_quads says that the list is not whole
    int slot = base + (int)incl - 1;  // the lane's slots are filled from its last one downwards
    const int dummy = CAP + lane;
    if (store) {  // uniform
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe(member, (uint32_t)(Q - 1 - q), 1u);  // all ones for a member
        const int to = (int)select_bits(m, (uint32_t)slot, (uint32_t)dummy);
        s.lists.quad[to] = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
        s.lists.id[to] = (uint32_t)(q << 16) | (uint32_t)tid;
        slot += (int)m;
      }
    }
  }
  listed();
  __syncthreads();
  const int n_quads = __builtin_amdgcn_readfirstlane(s.n_quads);
  if (n_quads > CAP || !store) return -1;

  // Step 3.
  for (int j0 = 0; j0 < n_quads; j0 += W * kWave) {
    if (j0 + wave * kWave >= n_quads) break;  // uniform over the wavefront
    const int j = j0 + tid;
    const bool live = j < n_quads;
    const float4 v = s.lists.quad[live ? j : 0];
    const uint32_t id = s.lists.id[live ? j : 0];
    const float e[4] = {v.x, v.y, v.z, v.w};
    bool keep[4];
    uint32_t n = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      keep[c] = live && keyof<NEG>(e[c]) >= T0;
      n += keep[c] ? 1u : 0u;
    }
    const uint32_t incl = wave_inclusive_scan_dpp(n);
    const int n_wave = __builtin_amdgcn_readlane((int)incl, kWave - 1);
    int base = 0;
    if (lane == 0) base = atomicAdd(&s.n_singles, n_wave);
    base = __builtin_amdgcn_readfirstlane(base);
    int at = base + (int)(incl - n);
    const int col = column((int)(id >> 16), (int)(id & 0xffffu));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (keep[c] && at < CAP) s.single[at] = make_uint2(__float_as_uint(e[c]), (uint32_t)(col + c));
      at += keep[c] ? 1 : 0;
    }
  }
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(s.n_singles);
  return n <= CAP ? n : -1;
}

// Steps 2 to 5 for one row, by the whole workgroup.  lo, hi: the keys' minimum and maximum; T0 the row's floor, probe
// see filter_search.  emit(place, value, column).  In the dense form nothing is emitted and thi, tlo, split say which
// elements stay: key >= (column <= split ? tlo : thi).  Every wavefront takes the same branches.
template <int E, int W, int ROOM, int MODE, bool NEG, int DT, bool DENSE, typename Column, typename Listed, typename Emit>
__device__ __forceinline__ int filter_row(FilterLds<W, ROOM>& s, const float (&x)[E], int lane, int wave, int k, int max_iter,
                                          float eps, float T0, float probe, float& lo, float& hi, float& thi, float& tlo,
                                          int& split, int& iterations, Column column, Listed listed, Emit emit) {
  constexpr int CAP = ROOM;
  constexpr bool BIG = ROOM > list_room(W);  // the bins, or no list
  const int tid = wave * kWave + lane;
  float low = lo;  // (lo itself stays for the caller's search of a row that the lists do not hold)
  int walked = 0;
  bool over = false;
  if constexpr (MODE != kExact) over = walk_to_floor<MODE>(T0, max_iter, eps, low, hi, walked);
  // (leaving before the lists are built costs the shape of 16 wavefronts about 90 spilled registers)
  int n = 0;
  if (W == 16 || !over) n = filter_lists<E, W, NEG>(s, x, lane, wave, T0, column, listed, !over);
  if (over) {
    lo = low;
    iterations = walked + 1;
    return kFilterBoundOnly;
  }
  if (n <= k) return kFilterNoList;  // (0 <= n <= k only with NaN or infinite keys)

  // Step 4 by wavefront 0, while every thread clears its words of the bitmaps.
  s.maps.cut[tid] = make_uint2(0u, 0u);
  s.maps.chosen[tid] = make_uint2(0u, 0u);
  if (wave == 0) {
    float l = low, h = hi, thres = low;
    bool hit = false;
    int steps = walked, cnt = -1, na = 0, last = 0x7fffffff;
    float by_bins_hi, by_bins_lo;
    int by_bins_limit = 0;
    bool found = false, ranked = false;
    if constexpr (MODE == kExact) {
      // (16-bit rows have few values, so a larger k finds many members in its bin: 2048 x 32768, bfloat16, k = 256, 256 rows
      // 10.4 -> 10.7 us with bins, k = 64 9.9 -> 9.3)
      if (BIG || DT == kF32 || k <= 128) {
        found = kth_by_bins<4, BIG ? 3 : 1, NEG>(s.single, n, lane, k, T0, hi, s.bins, by_bins_hi, by_bins_lo, last,
                                                 by_bins_limit);
      }
    } else if constexpr (BIG) {
      // the k-th key and the next, and the steps that they decide.  (On the shorter lists one wavefront counts a step in 150 cycles, and the ten
      // to twelve that end on a count of k cost less than bins and two passes: 64 x 16384, k = 250, 1e-4 10.4 -> 11.2 us, 16 steps 9.6 -> 11.0.)
      if (kth_by_bins<4, 3, NEG>(s.single, n, lane, k, T0, hi, s.bins, by_bins_hi, by_bins_lo, last, by_bins_limit)) {
        const float kth = by_bins_lo;
        float next;
        if (count_singles<NEG>(s.single, n, lane, kth, next) > k) next = kth;
        steps_by_rank<MODE>(kth, next, max_iter, eps, l, h, thres, hit, steps);
        cnt = hit ? k : -1;
        float unused;
        if (MODE == kEps && !hit) na = count_singles<NEG>(s.single, n, lane, h, unused);
        ranked = true;
      }
    }
    if (found || BIG) {
    } else if (n <= 4 * kWave) {
      filter_search<4, MODE, NEG, DT>(s.single, n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
    } else if (n <= 8 * kWave || CAP <= 8 * kWave) {
      filter_search<8, MODE, NEG, DT>(s.single, n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
    } else {
      filter_search<CAP / kWave, MODE, NEG, DT>(s.single, n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
    }
    // The selection as two thresholds and a limit: everything at or above t_hi, and of [t_lo, t_hi) the first `limit`
    // in column order (no limit: 0).
    const float inf = __builtin_inff();
    float t_hi, t_lo;
    int limit = 0;
    bool listed = true;
    if constexpr (MODE == kEarly) {
      t_lo = l;
      t_hi = cnt == k ? l : inf;
      limit = cnt == k ? 0 : k;
      listed = l >= T0;
    } else {
      if (found) {
        t_hi = by_bins_hi;
        t_lo = by_bins_lo;
        limit = by_bins_limit;
      } else if (hit) {
        t_hi = t_lo = thres;
      } else if (na >= k) {
        t_hi = inf;
        t_lo = h;
        limit = k;
      } else {
        t_hi = h;
        t_lo = l;
        limit = k - na;
        // exact mode has converged: [l, h) holds one value, which is on the list even where l is below the floor
        if constexpr (MODE == kEps) listed = l >= T0;
      }
    }
    if (lane == 0) {
      s.thr[0] = MODE == kEarly ? l : t_hi;  // the caller's selection, where the list has none, needs the bound itself
      s.thr[1] = t_lo;
      s.info[0] = limit;
      s.info[1] = hit ? steps : steps + 1;
      s.info[2] = found ? last : 0x7fffffff;
      s.state = (listed ? 0 : 1) | (MODE == kEarly && cnt != k ? 2 : 0) | (BIG && !found && !ranked ? 4 : 0);
    }
  }
  __syncthreads();
  const int state = __builtin_amdgcn_readfirstlane(s.state);
  tlo = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.thr[1])));
  thi = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.thr[0])));
  if (MODE == kEarly) thi = (state & 2) != 0 ? __builtin_inff() : thi;
  const int limit = __builtin_amdgcn_readfirstlane(s.info[0]);
  iterations = __builtin_amdgcn_readfirstlane(s.info[1]);
  split = MODE == kExact ? __builtin_amdgcn_readfirstlane(s.info[2]) : 0x7fffffff;
  if (BIG && (state & 4) != 0) return kFilterNoList;
  if ((state & 1) != 0) {
    lo = tlo;
    if (MODE == kEps) hi = thi;
    return kFilterBoundOnly;
  }

  // Step 5.  The cut class first, where there is one: the column of its limit-th member.
  if (limit > 0) {
    for (int j = tid; j < n; j += W * kWave) {
      const uint2 e = s.single[j];
      const float key = keyof<NEG>(__uint_as_float(e.x));
      if (key >= tlo && !(key >= thi)) atomicOr(reinterpret_cast<uint32_t*>(s.maps.cut) + (e.y >> 5), 1u << (e.y & 31));
    }
    __syncthreads();
    filter_prefix(s, s.maps.cut, lane, wave);
    for (int j = tid; j < n; j += W * kWave) {
      const uint2 e = s.single[j];
      const float key = keyof<NEG>(__uint_as_float(e.x));
      if (key >= tlo && !(key >= thi) && filter_rank(s, s.maps.cut, (int)e.y) == (uint32_t)(limit - 1)) s.info[2] = (int)e.y;
    }
    __syncthreads();
    split = __builtin_amdgcn_readfirstlane(s.info[2]);
  }
  if constexpr (!DENSE) {
    auto is_chosen = [&](const uint2& e) {
      return keyof<NEG>(__uint_as_float(e.x)) >= ((int)e.y <= split ? tlo : thi);
    };
    for (int j = tid; j < n; j += W * kWave) {
      const uint2 e = s.single[j];
      if (is_chosen(e)) atomicOr(reinterpret_cast<uint32_t*>(s.maps.chosen) + (e.y >> 5), 1u << (e.y & 31));
    }
    __syncthreads();
    filter_prefix(s, s.maps.chosen, lane, wave);
    for (int j = tid; j < n; j += W * kWave) {
      const uint2 e = s.single[j];
      if (is_chosen(e)) {
        const uint32_t place = filter_rank(s, s.maps.chosen, (int)e.y);
        if (place < (uint32_t)k) emit((int)place, e.x, (int)e.y);
      }
    }
  }
  return kFilterDone;
}

// ---- one wavefront per row ------------------------------------------------------------------------------
//
// The same for a row that one wavefront holds (16 to 128 values per lane).  Without other wavefronts to meet, both
// lists are kept in column order -- a quad's slot is the number of members in lower lanes and earlier groups (a lane
// mask's prefix count), a single's the scan of its quad's members -- so the winners' places are prefix counts too and no
// bitmap is needed.  The singles overwrite the quads that have been read.

// Group maxima per lane: 256 per row suffice for a small k; up to 55 % of them may lie above the floor, which then has
// 1.45 k candidates.  Twice as many for a larger k.
constexpr int wave_groups(int E, bool many) {
  return E <= 24 ? E / 4 : (!many ? 4 : (E == 48 ? 12 : 8));
}
constexpr int wave_filter_small_k(int E) { return 35 * wave_groups(E, false); }
// The largest k that takes the lists.  Beyond it a row's candidates fill eight registers of singles and more, and the LDS of
// the lists leaves fewer wavefronts in flight; 2^25 values, full-width search -> lists (us; exact mode): 1280 columns
// k = 140 43 -> 43, 175 43 -> 45; 2048 columns 175 31 -> 28, 245 30 -> 34; 3072 columns 245 31 -> 28, 280 31 -> 30, 420 31 -> 63
// (the lists never hold); 6146 columns 245 40 -> 33, 280 40 -> 46.  The dense form, bound by its stores, gains nothing
// from the lists and loses what wavefronts they cost: 8192 columns k = 64 47 -> 48, 140 50 -> 54, 280 51 -> 59.
// Rows of 16 values per lane: only the kernel of one row, see one_row_lists; the precision-bounded mode, whose trajectory
// starts at the row's minimum, keeps its full-width search there (k = 128 124 -> 135 us, 64 no difference).  Below 16 the
// full-width search costs no more than the lists do.
constexpr int wave_filter_max_k(int E, int R, int mode, bool dense = false) {
  if (R > 1 || E < (mode == kEps ? 24 : 16)) return 0;
  if (dense) return E <= 24 ? 100 : (E <= 64 ? 175 : 48);
  return E <= 24 ? 140 : (E == 32 ? 175 : 280);
}
// Whether a call takes them (uniform over the launch).  Above k = 245 only where k is at most 68 % of the row's group maxima: a
// row that leaves its layout a quarter empty has too few (k = 280: 4096 columns 33 -> 28 us, 3584 35 -> 34, 3074 40 -> 47).
// Algorithm 2 with few steps searches the full width: the last threshold of few steps lies below the floor, and each step
// saved is worth the less the narrower the row (1280 columns, bfloat16, five steps, k = 140: 38 -> 43 us, 100 38 -> 37).
// Rows of 16 values per lane, whose search over the row is short, are narrower still for their group maxima: k at most 74 % of
// these and fewer where four registers would not hold the singles; with fewer steps of Algorithm 2 less (one row per wavefront,
// 4096 / 30000 rows, search over the row -> lists: bfloat16 exact 514 columns, k = 90 10.8 / 36.9 -> 9.0 / 31.7, 110 10.8 / 37.5 -> 11.6 /
// 39.0; 600, k = 110 11.1 / 38.3 -> 9.4 / 32.8; 700, k = 130 11.2 / 39.0 -> 12.2 / 38.3; fp32 exact 770, k = 130 10.8 / 35.9 -> 9.8 / 34.6, 140
// 10.9 / 34.3 -> 12.2 / 39.3; eight steps 1000, k = 90 8.7 / 30.8 -> 8.4 / 29.6, 130 8.8 / 31.0 -> 9.1 / 32.4; six 131072 rows of 1000, k = 16
// 94.5 -> 91.2, 50000 rows, k = 64 42.6 -> 40.9; five 900, k = 64 6.8 / 24.1 -> 7.3 / 25.6; dense, 1000 rows of 770, k = 64 eight 5.7 -> 6.0,
// twelve 6.6 -> 6.1).  For the host, which tells the kernel: weighed there, the conditions cost the kernels of early stopping 3 to 11 %.
constexpr bool narrow_lists_hold(int mode, bool dense, int M, int k, int max_iter) {
  if (mode == kExact || max_iter >= 12) return 27 * k <= 5 * M && 14 * k <= M + 1064;
  if (max_iter >= 8) return (dense ? 16 : 8) * k <= M;
  return !dense && max_iter >= 6 && (max_iter == 7 ? 9 : 12) * k <= M;
}
__host__ __device__ constexpr bool wave_filter_takes(int E, int R, int mode, bool dense, int M, int k, int max_iter) {
  const int least = k > 245 ? 8 : (E <= 32 && k > 100 ? 6 : 5);
  return k <= wave_filter_max_k(E, R, mode, dense) && (k <= 245 || 100 * k * (E / wave_groups(E, true)) <= 68 * M) &&
         (mode != kEarly || max_iter >= least);
}
// What a launch says of it, and the kernel then knows (E = 16 by what it was told).
constexpr int kTakesLists = 4;  // a bit beside the kind of stores
inline int lists_flag(int E, int R, int mode, bool dense, int M, int k, int max_iter) {
  return E == 16 && k <= wave_filter_max_k(E, R, mode, dense) && narrow_lists_hold(mode, dense, M, k, max_iter) ? kTakesLists : 0;
}
__host__ __device__ constexpr bool takes_lists(int E, int R, int mode, bool dense, int M, int k, int max_iter, int flags) {
  return E == 16 ? R == 1 && (flags & kTakesLists) != 0 : wave_filter_takes(E, R, mode, dense, M, k, max_iter);
}
// Quads, and singles, that the lists of a row hold, and the pairs' worth of LDS they take.
__host__ __device__ constexpr int wave_filter_room(int k) { return (k + k / 2 + 48 + 63) & ~63; }
__host__ __device__ constexpr int wave_filter_pairs(int k) { return wave_filter_room(k) * 20 / 8; }

// One row.  x: masked elements; lo, hi: the keys' minimum and maximum; lists: wave_filter_pairs(k) pairs of LDS, 16-byte
// aligned; stage: where the pairs go (it may be the same memory).  In the dense form thi, tlo, split say which elements
// stay.  Returns a FilterResult.
template <int G, int NG, bool FULL, int MODE, bool NEG, int DT, bool DENSE>
__device__ __forceinline__ int filter_wave_row(const float (&x)[Layout<G, NG>::E], int lane, int M, int k, int max_iter,
                                               float eps, float& lo, float& hi, uint2* lists, uint2* stage, float& thi,
                                               float& tlo, int& split, int& iterations) {
  using L = Layout<G, NG>;
  constexpr int E = L::E;
  const int room = wave_filter_room(k);
  float4* quad = reinterpret_cast<float4*>(lists);
  uint32_t* id = reinterpret_cast<uint32_t*>(quad + room);  // first column of a quad

  float T0, probe;
  const int halvings = MODE == kEarly && max_iter <= 16 ? max_iter : 0;
  if (k <= wave_filter_small_k(E)) {  // uniform over the launch
    float gm[wave_groups(E, false)];
    lane_group_maxima<E, NEG>(x, gm);
    T0 = floor_of_maxima(gm, k + 1, lo, hi, probe, halvings);
  } else {
    float gm[wave_groups(E, true)];
    lane_group_maxima<E, NEG>(x, gm);
    T0 = floor_of_maxima(gm, k + 1, lo, hi, probe, halvings);
  }
  float low = lo;  // (lo itself stays for the caller's search of a row that the lists do not hold)
  int walked = 0;
  if constexpr (MODE != kExact) {
    if (walk_to_floor<MODE>(T0, max_iter, eps, low, hi, walked)) {
      lo = low;
      iterations = walked + 1;
      return kFilterBoundOnly;
    }
  }

  // quads with a key at or above the floor, in column order
  uint32_t nq = 0;  // wave-uniform
  static_for<L::GROUPS>([&](auto gc) {
    constexpr int g = decltype(gc)::value, e0 = L::first(g), H = L::width(g) / 4;
    int ln = lane;  // opaque per group, see compact_masks
    asm volatile("" : "+v"(ln));
    uint64_t m[H];
    uint32_t slot = nq;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int e = e0 + 4 * h;
      m[h] = __builtin_amdgcn_ballot_w64(key_max_on<NEG>(key_max3<NEG>(x[e], x[e + 1], x[e + 2]), x[e + 3]) >= T0);
      slot = lanes_below(m[h], slot);
    }
    const int col = group_col<G, NG, FULL>(g, ln, M);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int e = e0 + 4 * h;
      if (((m[h] >> lane) & 1) != 0 && slot < (uint32_t)room) {
        quad[slot] = make_float4(x[e], x[e + 1], x[e + 2], x[e + 3]);
        id[slot] = (uint32_t)(col + 4 * h);
      }
      nq += (uint32_t)__builtin_popcountll(m[h]);
      if (h + 1 < H) slot = add_mask_bit(slot, m[h]);
    }
    __builtin_amdgcn_sched_barrier(0);
  });
  if (nq > (uint32_t)room) return kFilterNoList;

  // their singles; a round's quads are in registers before it writes, and it writes no further than it has read
  uint32_t n = 0;
  for (uint32_t j0 = 0; j0 < nq; j0 += kWave) {
    const uint32_t j = j0 + (uint32_t)lane;
    const bool live = j < nq;
    const float4 v = quad[live ? j : 0];
    const uint32_t col = id[live ? j : 0];
    const float e[4] = {v.x, v.y, v.z, v.w};
    bool keep[4];
    uint32_t mine = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      keep[c] = live && keyof<NEG>(e[c]) >= T0;
      mine += keep[c] ? 1u : 0u;
    }
    const uint32_t incl = wave_inclusive_scan_dpp(mine);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    if (n + total > 2 * (j0 + kWave)) return kFilterNoList;  // uniform: 8 bytes each over quads of 16 already read
    uint32_t at = n + incl - mine;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (keep[c]) lists[at] = make_uint2(__float_as_uint(e[c]), col + (uint32_t)c);
      at += keep[c] ? 1u : 0u;
    }
    n += total;
  }
  constexpr int kMost = E <= 16 ? 4 : 8;  // registers of singles
  if (n <= (uint32_t)k || n > (uint32_t)(kMost * kWave)) return kFilterNoList;  // (n <= k only with NaN or infinite keys)

  float thres = low, l = low, h = hi;
  bool hit = false, found = false;
  int steps = walked, cnt = -1, na = 0, limit = 0;
  split = 0x7fffffff;
  if constexpr (MODE == kExact && DT == kF32) {
    // (the bins at the end of the lists' memory, where no single reaches)
    const int bytes = room * 20 - kBins * 4;
    uint32_t* bins = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(lists) + bytes);
    if ((int)n * 8 <= bytes && (E > 16 || k > 8 || DENSE)) found = kth_by_bins<1, 1, NEG>(lists, (int)n, lane, k, T0, hi, bins, thi, tlo, split, limit);
  }
  if (found) {
  } else if (n <= 2 * kWave) {
    filter_search<2, MODE, NEG, DT>(lists, (int)n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
  } else if (n <= 4 * kWave) {
    filter_search<4, MODE, NEG, DT>(lists, (int)n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
  } else if (kMost > 4) {
    filter_search<kMost, MODE, NEG, DT>(lists, (int)n, lane, k, max_iter, eps, T0, probe, l, h, thres, hit, steps, cnt, na);
  }
  // the selection as two thresholds and a limit, see filter_row
  iterations = hit ? steps : steps + 1;
  if constexpr (MODE == kEarly) {
    lo = l;
    if (!(l >= T0)) return kFilterBoundOnly;
    tlo = l;
    thi = cnt == k ? l : __builtin_inff();
    limit = cnt == k ? 0 : k;
  } else if (found) {
  } else if (hit) {
    thi = tlo = thres;
  } else if (na >= k) {
    thi = __builtin_inff();
    tlo = h;
    limit = k;
  } else {
    thi = h;
    tlo = l;
    limit = k - na;
    if (MODE == kEps && !(l >= T0)) {
      lo = l;
      hi = h;
      return kFilterBoundOnly;
    }
  }
  if (DENSE && limit == 0) return kFilterDone;

  // All singles go to registers before the first pair is staged: the stage may be the lists' memory.
  uint2 s[kMost];
#pragma unroll
  for (int i = 0; i < kMost; ++i) {
    if ((uint32_t)(i * kWave) < n) {  // uniform
      const uint32_t j = (uint32_t)(i * kWave + lane);
      s[i] = lists[j < n ? j : 0];
      if (j >= n) s[i].x = __float_as_uint(NEG ? __builtin_inff() : -__builtin_inff());
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint32_t stage_addr = (uint32_t)(uintptr_t)stage;
  uint32_t place = 0, in_band = 0;  // wave-uniform: chosen so far, members of the cut class so far
#pragma unroll
  for (int i = 0; i < kMost; ++i) {
    if ((uint32_t)(i * kWave) < n) {
      const float key = keyof<NEG>(__uint_as_float(s[i].x));
      uint64_t m = __builtin_amdgcn_ballot_w64(key >= (MODE == kExact && found && (int)s[i].y <= split ? tlo : thi));
      if (limit > 0) {  // uniform
        const uint64_t band = __builtin_amdgcn_ballot_w64(key >= tlo) & ~m;
        const uint64_t first = band & __builtin_amdgcn_ballot_w64(lanes_below(band, in_band) < (uint32_t)limit);
        in_band += (uint32_t)__builtin_popcountll(band);
        m |= first;
        if constexpr (DENSE) {
          if (first != 0) split = __builtin_amdgcn_readlane((int)s[i].y, 63 - __builtin_clzll(first));
        }
      }
      if constexpr (!DENSE) {
        const uint32_t pos = lanes_below(m, place);
        m &= __builtin_amdgcn_ballot_w64(pos < (uint32_t)k);  // (more than k only with NaN or infinite keys)
        lds_store_pair_masked(m, stage_addr + pos * 8u, s[i].x, s[i].y);
        place += (uint32_t)__builtin_popcountll(m);
      }
    }
  }
  return kFilterDone;
}
