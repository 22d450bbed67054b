// Rows of more than 32768 columns (fp32) spread over several workgroups, with scratch memory from the caller.
//
// One workgroup per row leaves the chip idle when there are few rows, and a row that fills a compute unit's register
// file by itself (32769 .. 65536 columns) leaves it idle while that row is searched.  Here a row is cut into segments of
// at most 32768 (or 16384, with longer lists up to 65536) columns, a workgroup each, in two launches:
//   rtopk_segment_kernel: every segment's candidates -- the keys at or above a floor with more than k keys of the segment
//     at or above it (steps 1 to 3 of rtopk_filter.hpp) -- go to the scratch memory in column order, with the floor and the
//     segment's minimum and maximum.  Where values crowd too much for the list (ties, sorted rows), the full-width search of
//     rtopk_block_kernel.hpp finds the segment's k + 1 largest keys instead, whose last is the floor: of the keys equal to it
//     the first in column order are listed, more than the row's selection can take from this segment;
//   rtopk_merge_kernel: one workgroup per row.  The largest of the segments' floors has more than k keys of the row at or
//     above it, and the lists hold all of those, so Algorithms 1 and 2 run on the lists with exact branch decisions (see
//     rtopk_filter.hpp; exact mode finds the k-th key by bins instead, and so do the others where they have steps enough, which
//     the k-th and the next key then decide without a count); the lists follow each other in column order, so
//     places are prefix counts.
// A row whose last threshold is not above the floor is written from the row itself.  A row with more candidates than the
// merging workgroup's registers hold (only where `cap` of split_of says that they may) is done by that workgroup as a
// streamed row (rtopk_stream_kernel.hpp).  Results are those of the other kernels.  Rows of more than 65536 columns whose k or whose
// number of segments is too large for that take longer lists, and a merge of more of them (split_big_of).
//
// What bounds it: the segments read the row once at the rate of the 32768-column rows (1.15 times the copy rate's time),
// the lists add 8 bytes per candidate written and read, 1.2 to 1.4 k of them per segment.  The merge is a launch and a chain of
// latencies, in which few wavefronts share a SIMD and each instruction takes one of them about seven cycles: so every wavefront finds
// its registers' lists from the heads by itself (a search for each candidate's list through LDS, behind a barrier, took 1 x 671792, k = 80, 41 lists,
// 13.7 us in all, 12.0 without; 64 x 131072 13.5 and 13.1), the loads are
// issued together, the fewest of 4, 8, 12, 16 or 40 registers that hold the row's candidates are walked, and exact mode counts each
// key into a bin once instead of in 10 to 14 steps of a barrier each (one row of 131072 columns, the merge alone: 7.8 -> 4 us).  Kernel
// time, one workgroup per row -> split with steps -> with bins: 64 x 131072, k = 50: 39.5 -> 19.2 -> 13.5 us; 1 x 131072: 36.5 -> 12.6 ->
// 8.7; 2048 x 50000, k = 100, registers of one workgroup -> split: 135 -> 88 -> 79; 16 x 2^20, k = 100: 31.0 -> 22.9;
// 256 x 262144, k = 512: 69 -> 59.
#pragma once

#include "rtopk_block_kernel.hpp"
#include "rtopk_stream_kernel.hpp"

namespace rtopk {

struct SegmentHead {
  int n;            // candidates
  float floor;      // every key of the segment at or above it is listed
  float nlo, hi;    // negated minimum, and maximum, of the segment's keys
};
static_assert(sizeof(SegmentHead) == kSegmentHeadBytes, "split_of counts it");

template <int NG, int W, bool NEG, bool BIG>
__global__ void __launch_bounds__(W * kWave) __attribute__((amdgpu_waves_per_eu(BIG ? 4 : 5)))
    rtopk_segment_kernel(const float* __restrict__ in, int M, int k, int segments, int length, int cap,
                         SegmentHead* __restrict__ heads, uint2* __restrict__ lists, uint32_t shares, uint32_t shares_last) {
  constexpr int G = 4, E = G * NG;
  __shared__ BoundsLds<W> s_bounds;
  __shared__ FilterLds<W, BIG ? kBigRoom : segment_room(W)> s_filter;
  const int lane = threadIdx.x & (kWave - 1), tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = (int)blockIdx.x / segments, seg = (int)blockIdx.x % segments;
  const int first = seg * length, cols = M - first < length ? M - first : length;  // at least G columns (split_of)
  const float* from = in + (int64_t)r * M + first;
  float x[E];
  block_load<kF32, G, W, 0, NG>(from, cols, lane, wave, x);
  int need = floor_share(cols, G, W, wave, cols < length ? shares_last : shares);
  asm volatile("" : "+s"(need));  // here, while the loads are in flight
  const float nm = lane_negmin<E, NEG>(x);
  block_mask<G, NG, W, NEG>(x, cols, lane, wave);
  if (tid == 0) {
    s_filter.n_quads = 0;
    s_filter.n_singles = 0;
  }
  float lo, hi, T0, probe;
  block_bounds<E, W, NEG, true, floor_groups(E, BIG)>(x, nm, need, lane, wave, s_bounds, lo, hi, T0, probe);
  auto column = [&](int quad, int thread) -> int { return min((quad * W * kWave + thread) * G, cols - G); };
  const int n = filter_lists<E, W, NEG>(s_filter, x, lane, wave, T0, column, [] {});
  uint2* to = lists + (int64_t)blockIdx.x * cap;
  if (n < 0 || n > cap) {  // uniform
    bool none = false;
    float ahead[block_groups_ahead(W, G, kFullWidth) * G + 1];
    KnownBounds end{};
    // (their values to the first half of the list's memory, their columns to the second; then in pairs like any other list)
    float* values = reinterpret_cast<float*>(to);
    int32_t* columns = reinterpret_cast<int32_t*>(to) + cap;
    block_row<G, NG, W, kExact, NEG, kF32, false, kFullWidth>(0, from, 1, cols, k + 1, 0, 0.0f, values, columns, nullptr, 0, 1,
                                                              none, ahead, none, x, end);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (it stores through inline asm)
    __syncthreads();
    constexpr int kMost = ((BIG ? kBigMaxK : filter_max_k(W)) + W * kWave) / (W * kWave);  // pairs per thread, k + 1 in all
    uint2 pair[kMost];
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      const int j = min(i * W * kWave + tid, k);
      pair[i] = make_uint2(__float_as_uint(values[j]), (uint32_t)(columns[j] + first));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      if (i * W * kWave + tid <= k) to[i * W * kWave + tid] = pair[i];
    }
    if (tid == 0) heads[blockIdx.x] = SegmentHead{k + 1, end.lo, -lo, hi};
    return;
  }
  if (tid == 0) heads[blockIdx.x] = SegmentHead{n, T0, -lo, hi};
  // in column order: the places of the singles' bits
  s_filter.maps.chosen[tid] = make_uint2(0u, 0u);
  __syncthreads();
  for (int j = tid; j < n; j += W * kWave) {
    const uint32_t c = s_filter.single[j].y;
    atomicOr(reinterpret_cast<uint32_t*>(s_filter.maps.chosen) + (c >> 5), 1u << (c & 31));
  }
  __syncthreads();
  filter_prefix(s_filter, s_filter.maps.chosen, lane, wave);
  for (int j = tid; j < n; j += W * kWave) {
    const uint2 e = s_filter.single[j];
    const uint32_t place = filter_rank(s_filter, s_filter.maps.chosen, (int)e.y);
    if (place < (uint32_t)n) to[place] = make_uint2(e.x, e.y + (uint32_t)first);  // (NaN keys could share a column's bit)
  }
}

// What the search of a row leaves to be written from the row itself: two classes of keys and a limit for each (as in
// rtopk_block_kernel.hpp).
struct RowClasses {
  float tA, tB;
  int limA, limB;
};
enum MergeResult : int {
  kMergeDone = 0,     // the pairs are written
  kMergeNoList = 1,   // the lists do not hold the search
  kMergeFromRow = 2   // the search is over; the selection reaches below the floor
};

template <int NW>
struct MergeLds {
  int first[kMaxSegments + 1];  // candidates in earlier segments
  float bound[3];
  int total, cnt[2][NW], cls[2][NW];
  alignas(16) uint32_t bins[kBins];
  uint2 member[kWave];  // of the bin with the k-th key: (key bits, column), any order
  uint32_t members;
  float below[NW];  // per wavefront: its largest key in lower bins
};

// One row's candidates, KR registers of them per lane, `per` in use.  All loads are issued together, of 40 registers eight at a
// time, with 32-bit offsets: a row's lists are less than 2 GiB.
//
// By lists, up to 64 of them: a register holds 64 consecutive candidates of one list, so what it loads is the same for all lanes: lane s
// knows where list s starts among the registers of the row (`start`), and the list of a register is the number of lanes that start at or
// before it.  key = NaN (at or above no threshold) behind a list's end.
template <int NW, int KR, bool NEG>
__device__ __forceinline__ void load_by_lists(const uint2* __restrict__ lists, int segments, int cap, int start, int n, int per,
                                              float (&key)[KR], uint32_t (&col)[KR]) {
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  constexpr int kBatch = KR <= 16 ? KR : 8;
  auto load = [&](auto from) {
    constexpr int I0 = decltype(from)::value * kBatch;
    uint2 v[kBatch];
    int left[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int u = wave * per + I0 + i;
      const int seg = max(__builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < segments && start <= u)) - 1, 0);
      const int first = (u - __builtin_amdgcn_readlane(start, seg)) * kWave;  // beyond the last list's end where there are no more
      left[i] = I0 + i < per ? __builtin_amdgcn_readlane(n, seg) - first : 0;
      const uint32_t at = (uint32_t)(seg * cap + (left[i] > 0 ? first + min(lane, left[i] - 1) : 0));
      v[i] = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(lists) + at * 8u);
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      key[I0 + i] = lane < left[i] ? keyof<NEG>(__uint_as_float(v[i].x)) : __builtin_nanf("");
      col[I0 + i] = v[i].y;
    }
  };
  static_for<KR / kBatch>(load);
}
// By number, 64 consecutive ones of the row to a register: number wave * per * 64 + i * 64 + lane (a lane beyond the last candidate
// repeats its load); s.first: candidates in earlier lists.
template <int NW, int KR, bool NEG>
__device__ __forceinline__ void load_by_number(const MergeLds<NW>& s, const uint2* __restrict__ lists, int segments, int cap, int per,
                                               int total, float (&key)[KR], uint32_t (&col)[KR]) {
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  constexpr int kBatch = KR <= 16 ? KR : 8;  // (more of them would not fit beside the 40 registers of the largest)
  const int top = segments > 1 ? 1 << (31 - __builtin_clz(segments - 1)) : 0;
  auto load = [&](auto from) {
    constexpr int I0 = decltype(from)::value * kBatch;
    int seg[kBatch], e[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      seg[i] = 0;  // the last segment that starts at or before the candidate and is not empty
      e[i] = min((wave * per + I0 + i) * kWave + lane, total - 1);
    }
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int next = min(seg[i] + step, segments);
        seg[i] = s.first[next] <= e[i] ? next : seg[i];
      }
    }
    uint2 v[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const uint32_t at = (uint32_t)(seg[i] * cap + e[i] - s.first[seg[i]]);
      v[i] = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(lists) + at * 8u);
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const bool live = I0 + i < per && (wave * per + I0 + i) * kWave + lane < total;
      key[I0 + i] = live ? keyof<NEG>(__uint_as_float(v[i].x)) : __builtin_nanf("");  // (at or above no threshold)
      col[I0 + i] = v[i].y;
    }
  };
  static_for<KR / kBatch>(load);
}

// The search and the pairs from the candidates in registers (in column order: by wavefront, register and lane).  Bins and members
// are cleared and a barrier has passed.  Uniform over the workgroup.
template <int NW, int KR, int MODE, bool NEG, bool RANK>
__device__ __forceinline__ MergeResult merge_candidates(MergeLds<NW>& s, int64_t r, int M, int k, int max_iter, float eps_rel,
                                                        float* __restrict__ ov, int32_t* __restrict__ oi,
                                                        int32_t* __restrict__ out_iters, float (&key)[KR], uint32_t (&col)[KR],
                                                        int per, float T0, float lo, float hi, RowClasses& rest) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // RANK: the k-th key by bins (see kth_by_bins): every wavefront bins its own, then all find the same bin and rank its members.
  // Exact mode takes the keys above it and the first of those equal to it; the other modes' steps are decided by it and
  // the next one (steps_by_rank).
  bool ranked = false;
  float kth = 0.0f, next = 0.0f;
  const float eps = MODE == kEps ? eps_rel * __builtin_fabsf(hi) : 0.0f;
  // (not where the steps hardly reach the floor, as from a mask's -1e9: 1 x 65860, k = 76, 16 steps 12.5 us, ranked first 13.4)
  const float last_width = MODE == kEarly ? __builtin_ldexpf(hi - lo, -max_iter) : eps;
  if (RANK && (MODE == kExact || last_width * 16.0f < hi - T0)) {  // uniform
    const float scale = bins_scale(T0, hi);
#pragma unroll
    for (int i = 0; i < KR; ++i) {
      if (key[i] >= T0) atomicAdd(&s.bins[bin_of(key[i], hi, scale)], 1u);
    }
    __syncthreads();
    int above, in_bin;
    const int chosen = find_bin(s.bins, lane, k, above, in_bin);
    if (chosen >= 0 && in_bin <= kWave) {  // uniform
      const bool last_in_bin = MODE != kExact && k - above == in_bin;  // the next key is in a lower bin
      float below = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < KR; ++i) {
        if constexpr (KR > 16) asm volatile("" : "+v"(key[i]));  // (the bins are not kept in as many registers again)
        if (key[i] >= T0) {
          const int bin = bin_of(key[i], hi, scale);
          if (bin == chosen) {
            const uint32_t at = atomicAdd(&s.members, 1u);
            if (at < (uint32_t)kWave) s.member[at] = make_uint2(__float_as_uint(key[i]), col[i]);
          }
          if (MODE != kExact && bin > chosen) below = vmax(below, key[i]);
        }
      }
      if (last_in_bin) {  // uniform
        float largest, unused;
        wave_max_and_negmin(below, below, largest, unused);
        if (lane == 0) s.below[wave] = largest;
      }
      __syncthreads();
      int tcol;
      bool cut;
      ranked = rank_members<MODE != kExact>(s.member, lane, in_bin, k - above, kth, tcol, cut, next);
      if (last_in_bin) {
#pragma unroll
        for (int w = 0; w < NW; ++w) next = w == 0 ? s.below[0] : vmax(next, s.below[w]);
        ranked = ranked && next > -__builtin_inff();
      }
      if (MODE == kExact && ranked) {
        auto chosen_mask = [&](int i) -> uint64_t {
          return __builtin_amdgcn_ballot_w64(key[i] > kth || (key[i] == kth && (int)col[i] <= tcol));
        };
        constexpr bool kKeep = KR <= 16;
        uint64_t kept[kKeep ? KR : 1];
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < KR; ++i) {
          const uint64_t m = chosen_mask(i);
          if constexpr (kKeep) kept[i] = m;
          mine += (uint32_t)__builtin_popcountll(m);
        }
        if (lane == 0) s.cls[0][wave] = (int)mine;
        __syncthreads();
        uint32_t place = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) place += w < wave ? (uint32_t)s.cls[0][w] : 0u;
#pragma unroll
        for (int i = 0; i < KR; ++i) {
          if constexpr (!kKeep) asm volatile("" : "+v"(key[i]));
          uint64_t m;
          if constexpr (kKeep) m = kept[i]; else m = chosen_mask(i);
          const uint32_t at = lanes_below(m, place);
          if (((m >> lane) & 1) != 0 && at < (uint32_t)k) {
            ov[at] = keyof<NEG>(key[i]);
            oi[at] = (int32_t)min(col[i], (uint32_t)(M - 1));  // (NaN keys can leave list entries unwritten)
          }
          place += (uint32_t)__builtin_popcountll(m);
        }
        return kMergeDone;
      }
    }
  }
  int turn = 0;
  auto count = [&](float t) -> int {  // one barrier; the halves of s.cnt alternate as in rtopk_block_kernel
    int mine = 0;
#pragma unroll
    for (int i = 0; i < KR; ++i)
      if (i < per) mine += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >= t));
    const int p = turn & 1;
    ++turn;
    if (lane == 0) s.cnt[p][wave] = mine;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane((int)row16_sum(lane < NW ? (uint32_t)s.cnt[p][lane] : 0u));
  };
  bool hit = false;
  float thres = lo;
  int steps = 0;
  if (RANK && MODE != kExact && ranked) {
    steps_by_rank<MODE>(kth, next, max_iter, eps, lo, hi, thres, hit, steps);
  } else {
    if (count(T0) <= k) return kMergeNoList;  // (only with NaN or infinite keys)
    // The search (see filter_search): exact mode may start at the floor, the others follow their thresholds.
    if (MODE == kExact) lo = T0;
    for (;;) {
      if (MODE == kEarly && steps >= max_iter) break;
      if (MODE == kEps && !(hi - lo > eps)) break;
      const float mid = (lo + hi) * 0.5f;
      if (!(mid > lo && mid < hi)) {
        // no fp32 value strictly inside (lo, hi): Algorithm 1 ends; Algorithm 2's steps repeat one midpoint, equal to lo
        // (nothing moves) or to hi (lo moves up to it where hi itself counts k or more)
        if (MODE == kEarly && mid == hi && hi > lo && count(hi) >= k) lo = hi;
        break;
      }
      const int cnt = mid > T0 ? count(mid) : k + 1;
      thres = mid;
      ++steps;
      if (cnt == k) {
        hit = true;
        if (MODE == kEarly) lo = mid;
        break;
      }
      if (cnt < k) hi = mid; else lo = mid;
    }
  }
  // Two classes and a limit for each (as in rtopk_block_kernel).
  float tA, tB = 0.0f;
  int limA = k, limB = 0;
  if (MODE == kEarly) {
    tA = lo;
  } else if (hit) {
    tA = thres;
  } else {
    const int na = count(hi);
    tA = hi;
    tB = lo;
    limA = na < k ? na : k;
    limB = k - limA;
  }
  if constexpr (MODE == kEps) {
    if (out_iters != nullptr && tid == 0) out_iters[r] = hit ? steps : steps + 1;
  }
  // (At the floor itself a list may hold some of the keys only.  They are those that exact mode needs, whose class B is one
  // value; the other modes take the first keys of a whole range.)
  if (MODE != kExact && !((limB > 0 ? tB : tA) > T0)) {
    rest = RowClasses{tA, tB, limA, limB};
    return kMergeFromRow;
  }

  uint32_t nA = 0, nB = 0;
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    if (i < per) {
      nA += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >= tA));
      if (limB > 0) nB += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >= tB && !(key[i] >= tA)));
    }
  }
  if (lane == 0) {
    s.cls[0][wave] = (int)nA;
    s.cls[1][wave] = (int)nB;
  }
  __syncthreads();
  uint32_t posA0 = 0, posB0 = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    posA0 += w < wave ? (uint32_t)s.cls[0][w] : 0u;
    posB0 += w < wave ? (uint32_t)s.cls[1][w] : 0u;
  }
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    if (i < per) {
      const bool a = key[i] >= tA, b = limB > 0 && key[i] >= tB && !a;
      const uint64_t mA = __builtin_amdgcn_ballot_w64(a), mB = __builtin_amdgcn_ballot_w64(b);
      const uint32_t posA = lanes_below(mA, posA0), posB = lanes_below(mB, posB0);
      if ((a && posA < (uint32_t)limA) || (b && posB < (uint32_t)limB)) {
        const uint32_t pos = (posA < (uint32_t)limA ? posA : (uint32_t)limA) + (posB < (uint32_t)limB ? posB : (uint32_t)limB);
        ov[pos] = keyof<NEG>(key[i]);
        oi[pos] = (int32_t)min(col[i], (uint32_t)(M - 1));  // (NaN keys can leave list entries unwritten)
      }
      posA0 += (uint32_t)__builtin_popcountll(mA);
      posB0 += (uint32_t)__builtin_popcountll(mB);
    }
  }
  return kMergeDone;
}

// Registers that a lane of NW merging wavefronts walks when it holds `per` candidates (the fewest that serve: a wavefront issues an instruction in
// seven cycles, and few share a SIMD here).
template <int NW>
__device__ __forceinline__ int registers_walked(int per, bool lists) {
  return per <= 4 ? 4 : (per <= 8 ? 8 : (lists && NW < 16 && per <= 12 ? 12 : (NW < 16 || per <= kMergeRegs ? kMergeRegs : kMergeRegsBig)));
}

// One row: its search on the segments' lists, and its selection from them, or, where the search ends on a minimum below
// the floor, from the row.  Returns false, with nothing written, where the lists do not hold the search.  Called by the
// whole workgroup; uniform.
template <int NW, int MODE, bool NEG, bool RANK>
__device__ __forceinline__ bool merge_row(MergeLds<NW>& s, int64_t r, const float* __restrict__ in, int M, int k, int max_iter,
                                          float eps_rel, float* __restrict__ out_vals, int32_t* __restrict__ out_idx,
                                          int32_t* __restrict__ out_iters, const SegmentHead* __restrict__ heads,
                                          const uint2* __restrict__ lists, int segments, int cap, int by_lists) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (RANK && wave == NW - 1) {
    clear_bins(s.bins, lane);
    if (lane == 0) s.members = 0;
  }
  float* ov = out_vals + r * (int64_t)k;
  int32_t* oi = out_idx + r * (int64_t)k;
  const uint2* of_row = lists + r * segments * cap;
  RowClasses rest;
  MergeResult done;
  constexpr int kMost = NW == 16 ? kMergeRegsBig : kMergeRegs;
  bool by_number = !by_lists;
  if (!by_number) {  // uniform
    // every wavefront reads the heads, lane s that of segment s: nothing to exchange before the bins
    const SegmentHead h = heads[r * segments + min(lane, segments - 1)];
    const int n = lane < segments ? h.n : 0, regs = (n + kWave - 1) / kWave;
    static_assert(kWave * kBigRoom < 1 << 17, "the candidates of 64 lists beside their registers");
    const uint32_t upto = wave_inclusive_scan_dpp((uint32_t)regs << 17 | (uint32_t)n);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
    const int start = (int)(upto >> 17) - regs;
    float T0, lo, hi, unused;
    wave_max_and_negmin(h.floor, h.nlo, T0, lo);  // (a lane beyond the last segment repeats it)
    wave_max_and_negmin(h.hi, h.hi, hi, unused);
    const int total = (int)(all & 0x1ffffu), per = ((int)(all >> 17) + NW - 1) / NW;
    auto listed = [&](auto regs_of) -> MergeResult {
      constexpr int KR = decltype(regs_of)::value;
      float key[KR];
      uint32_t col[KR];
      load_by_lists<NW, KR, NEG>(of_row, segments, cap, start, n, per, key, col);
      __syncthreads();
      return merge_candidates<NW, KR, MODE, NEG, RANK>(s, r, M, k, max_iter, eps_rel, ov, oi, out_iters, key, col, per, T0, lo, hi, rest);
    };
    // (lists of a few more than 64, 128 ... candidates leave most of a register empty: numbered through, half the registers may do.  By lists -> by number,
    // us: 40 registers to 16, 1 x 10^6, k = 700 37.3 -> 27.2; 16 to 8, k = 80 15.6 -> 14.3; 8 to 4, 16 wavefronts, 1 x 538928, k = 173 -8 %; exact mode,
    // 14 x 132306, k = 47 -3 %.  But 12 to 8, 1 x 311414, k = 134 13.4 -> 14.0, and 8 to 4 in few wavefronts, whose bins are not needed, 6 x 155042, k = 51,
    // eight steps 10.6 -> 10.9: then what the lists' places in LDS and the search for them cost is as much.)
    by_number = per > kMost || (per > (NW == 16 || MODE == kExact ? 4 : 12) &&
                                registers_walked<NW>(per, true) >= 2 * registers_walked<NW>((total + NW * kWave - 1) / (NW * kWave), false));
    if (by_number) {
      if (wave == 0) {
        if (lane < segments) s.first[lane] = (int)(upto & 0x1ffffu) - n;
        if (lane == 0) {
          s.first[segments] = s.total = total;
          s.bound[0] = T0;
          s.bound[1] = lo;
          s.bound[2] = hi;
        }
      }
    } else if (per <= 4) {
      done = listed(std::integral_constant<int, 4>());
    } else if (per <= 8) {
      done = listed(std::integral_constant<int, 8>());
    } else if (NW < 16 && per <= 12) {
      done = listed(std::integral_constant<int, NW < 16 ? 12 : 8>());
    } else if (NW < 16 || per <= kMergeRegs) {
      done = listed(std::integral_constant<int, kMergeRegs>());
    } else {
      done = listed(std::integral_constant<int, kMost>());
    }
  } else if (wave == 0) {
    float fl = -__builtin_inff(), nlo = -__builtin_inff(), top = -__builtin_inff();
    int before = 0;
    for (int s0 = 0; s0 < segments; s0 += kWave) {
      const bool live = s0 + lane < segments;
      const SegmentHead h = heads[r * segments + (live ? s0 + lane : 0)];
      const int n = live ? h.n : 0;
      const uint32_t incl = wave_inclusive_scan_dpp((uint32_t)n);
      if (live) s.first[s0 + lane] = before + (int)incl - n;
      before += __builtin_amdgcn_readlane((int)incl, kWave - 1);
      fl = vmax(fl, h.floor);  // (a lane beyond the last segment repeats the first)
      nlo = vmax(nlo, h.nlo);
      top = vmax(top, h.hi);
    }
    float a, b, c, unused;
    wave_max_and_negmin(fl, nlo, a, b);
    wave_max_and_negmin(top, top, c, unused);
    if (lane == 0) {
      s.first[segments] = before;
      s.total = before;
      s.bound[0] = a;
      s.bound[1] = b;
      s.bound[2] = c;
    }
  }
  if (by_number) {  // uniform
    __syncthreads();
    const int total = __builtin_amdgcn_readfirstlane(s.total);
    const float T0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.bound[0])));
    const float lo = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.bound[1])));
    const float hi = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.bound[2])));
    if (total <= k || total > NW * kWave * kMost) return false;
    const int per = (total + NW * kWave - 1) / (NW * kWave);
    auto numbered = [&](auto regs_of) -> MergeResult {
      constexpr int KR = decltype(regs_of)::value;
      float key[KR];
      uint32_t col[KR];
      load_by_number<NW, KR, NEG>(s, of_row, segments, cap, per, total, key, col);
      return merge_candidates<NW, KR, MODE, NEG, RANK>(s, r, M, k, max_iter, eps_rel, ov, oi, out_iters, key, col, per, T0, lo, hi, rest);
    };
    if (per <= 4) {  // (1 x 2200003, 135 lists: k = 10 19.7 us in 16 registers, 12.9 in 4; k = 20 20.1 and 15.3; 1 x 2^20, k = 8, four steps 16.3 and 11.5)
      done = numbered(std::integral_constant<int, 4>());
    } else if (per <= 8) {
      done = numbered(std::integral_constant<int, 8>());
    } else if (NW < 16 || per <= kMergeRegs) {
      done = numbered(std::integral_constant<int, kMergeRegs>());
    } else {
      done = numbered(std::integral_constant<int, kMost>());
    }
  }
  if (MODE != kExact && done == kMergeFromRow)  // (latency bound: a barrier per chunk; 16 wavefronts have the registers for four loads each)
    write_by_chunks<NW, 4, NEG, NW == 16 ? 4 : 2>(in + r * (int64_t)M, M, k, rest.tA, rest.tB, rest.limA, rest.limB, ov, oi);
  return done != kMergeNoList;
}

template <int NW, int MODE, bool NEG, bool RANK>
__global__ void __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(4)))
    rtopk_merge_kernel(const float* __restrict__ in, int M, int k, int max_iter, float eps_rel,
                       float* __restrict__ out_vals, int32_t* __restrict__ out_idx, int32_t* __restrict__ out_iters,
                       const SegmentHead* __restrict__ heads, const uint2* __restrict__ lists, int segments, int cap,
                       int by_lists) {
  const int64_t r = blockIdx.x;
  __shared__ union {
    MergeLds<NW> merge;
    StreamLds<NW> stream;
  } s;
  if (merge_row<NW, MODE, NEG, RANK>(s.merge, r, in, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters, heads, lists, segments, cap,
                                        by_lists)) return;
  __syncthreads();
  stream_row<NW, 4, MODE, NEG>(s.stream, r, in, M, k, max_iter, eps_rel, out_vals, out_idx, out_iters);
}

// Whether the merge finds the k-th key, from which every step follows, rather than count in each step.  Exact mode always; the other
// modes from about eight steps above the lists' floor on (us, steps counted -> by rank: precision 1e-6 36 x 63680, k = 82 14.1 -> 13.0, 1e-4
// 64 x 50000, k = 200 16.1 -> 15.0, 1e-2 14.0 -> 14.2; 64 x 50000 40 steps 16.0 -> 14.4, 16 15.5 -> 14.2, 8 13.2 -> 13.5; 8 x 10^6, k = 300, 16
// 28.1 -> 26.2), but not the longest lists, whose bins hold many (16 x 131072, k = 900, 16 steps 21.0 -> 21.8).
inline bool ranks(const Split& s, int mode, const LaunchArgs& a) {
  return mode == kExact || (!s.big && (mode == kEarly ? a.max_iter >= 12 : a.eps_rel < 0x1p-10f));
}
// Lists of less than half a register each are better numbered through (four wavefronts' floors leave 26 candidates at k = 8, 38 at 17; 2 x
// 655360, k = 8, 40 lists: by number 10.6 us, by lists 12.2; 2 x 983040, k = 17, 60 lists 11.8 and 10.9).
template <int MODE, bool NEG, bool RANK>
hipError_t launch_merge(const Split& s, int64_t rows, const SegmentHead* heads, const uint2* lists, const LaunchArgs& a, int64_t r0) {
  const bool by_lists = s.segments <= kWave && (s.w > 4 || a.k >= 16 || s.segments <= 8);
  const auto merge = s.merge_waves == 4   ? &rtopk_merge_kernel<4, MODE, NEG, RANK>
                     : s.merge_waves == 8 ? &rtopk_merge_kernel<8, MODE, NEG, RANK>
                                          : &rtopk_merge_kernel<16, MODE, NEG, RANK>;
  return launch_kernel(merge, dim3((unsigned)rows), dim3(s.merge_waves * kWave), 0, a.stream, static_cast<const float*>(a.in) + r0 * a.M,
                       a.M, a.k, a.max_iter, a.eps_rel, static_cast<float*>(a.out_vals) + r0 * a.k,
                       static_cast<int32_t*>(a.out_idx) + r0 * a.k, a.out_iters ? a.out_iters + r0 : nullptr, heads, lists, s.segments,
                       s.cap, by_lists ? 1 : 0);
}

template <int MODE, bool NEG>
hipError_t launch_split(const Split& s, void* scratch, const LaunchArgs& a) {
  const uint32_t shares = floor_shares(s.length, a.k, 4), shares_last = floor_shares(a.M - (s.segments - 1) * s.length, a.k, 4);
  for (int64_t r0 = 0; r0 < a.N; r0 += s.rows) {
    const int64_t rows = a.N - r0 < s.rows ? a.N - r0 : s.rows;
    const float* in = static_cast<const float*>(a.in) + r0 * a.M;
    SegmentHead* heads = static_cast<SegmentHead*>(scratch);
    uint2* lists = reinterpret_cast<uint2*>(heads + rows * s.segments);
    const auto segment = s.big      ? (s.w == 8 ? &rtopk_segment_kernel<16, 8, NEG, true> : &rtopk_segment_kernel<16, 16, NEG, true>)
                         : s.w == 4 ? (s.ng == 12 ? &rtopk_segment_kernel<12, 4, NEG, false> : &rtopk_segment_kernel<16, 4, NEG, false>)
                                    : (s.ng == 12 ? &rtopk_segment_kernel<12, 8, NEG, false> : &rtopk_segment_kernel<16, 8, NEG, false>);
    hipError_t err = launch_kernel(segment, dim3((unsigned)(rows * s.segments)), dim3(s.w * kWave), 0, a.stream, in, a.M, a.k,
                                   s.segments, s.length, s.cap, heads, lists, shares, shares_last);
    if (err != hipSuccess) return err;
    hipError_t (*const merge)(const Split&, int64_t, const SegmentHead*, const uint2*, const LaunchArgs&, int64_t) =
        ranks(s, MODE, a) ? &launch_merge<MODE, NEG, true> : &launch_merge<MODE, NEG, MODE == kExact>;
    err = merge(s, rows, heads, lists, a, r0);
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace rtopk
