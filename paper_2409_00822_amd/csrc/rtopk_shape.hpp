// Shape classification of the row-wise top-k library: which kernel family and which register layout a
// call's row width, element type and pointer alignment map to.  Host code only (no HIP headers), so that
// it can also be compiled and swept by a CPU test under the address / undefined-behaviour sanitizers.
//
// A layout is (g, ng, w): a lane owns ng groups of g consecutive columns, and a row is spread over w
// wavefronts (w = 1: one wavefront per row, rtopk_kernel.hpp; w > 1: one workgroup per row,
// rtopk_block_kernel.hpp), so a layout holds rows of up to 64 * g * ng * w columns.
//
// The kernels load vectors from any element boundary at full rate, so what counts is only how little of a lane's
// registers a row leaves empty: kernel_layout() goes by width, type and form, not by alignment.  Which layouts
// are compiled is fixed by the lists below; the instantiation tables (rtopk_inst_*.hip) expand the same lists, so a
// layout that kernel_layout() returns always has a kernel behind it.
#pragma once

#include <stdint.h>

// Groups per lane that are instantiated, per load width.  X(n) is expanded once per entry, ascending.
#define RTOPK_NG_LIST_G4(X) X(1) X(2) X(3) X(4) X(6) X(8) X(12) X(16) X(24) X(32)   /* fp32, 128-bit loads */
#define RTOPK_NG_LIST_H8(X) X(1) X(2) X(3) X(4) X(6) X(8) X(12) X(16)               /* 16-bit rows, 128-bit loads */
// Rows of up to 448 columns, X(g, ng): one or two values per lane, and (g = 0) three, five, six or seven in
// groups of mixed width (Layout in rtopk_kernel.hpp); four are (4, 1) of the lists above, eight (4, 2) or (8, 1).
#define RTOPK_LAYOUT_LIST_SMALL(X) X(1, 1) X(2, 1) X(0, 3) X(0, 5) X(0, 6) X(0, 7)

namespace rtopk {

// Which algorithm of the paper (Section 3.1) a kernel instance runs.
enum Mode : int {
  kEarly = 0,  // Algorithm 2: max_iter steps, one-pass selection against min
  kExact = 1,  // Algorithm 1 at epsilon = 0
  kEps = 2     // Algorithm 1 with epsilon = eps_rel * |max|, optional exit-iteration output
};

// Element type of the input matrix and of the value output.
enum DType : int {
  kF32 = 0,
  kF16 = 1,  // IEEE half
  kBF16 = 2  // bfloat16
};

constexpr int kMaxM = 1 << 24;       // widest row at all (fp32 rows, int32 columns: streamed beyond kMaxBlockM)
constexpr int kMaxBlockM = 65536;    // widest row one workgroup holds in registers; the limit of the 16-bit and dense forms
constexpr int kMaxWaveM = 8192;      // widest row one wavefront holds in registers
constexpr int kBackwardRowsM = 2048;  // backward edge: widest row assembled whole in a wavefront's LDS (8 KiB)

enum Family : int {
  kFamSmall = 0,  // launch_small_*: fp32 rows of up to 448 columns whose lanes do not hold exactly four values
  kFamG4 = 1,     // launch_g4_*: fp32, 128-bit loads
  kFamH16 = 2,    // launch_h16_*: half / bfloat16 rows, one wavefront per row
  kFamBlock = 3,  // launch_block_*: one workgroup per row, the row in registers
  kFamStream = 4  // launch_stream: one workgroup per row, the row streamed several times (fp32, int32 columns)
};

struct Shape {
  int family;
  int g, ng, w;  // g = 0: groups of mixed width, ng values per lane
  bool full;     // M == 64 * g * ng * w: the kernel needs no column-validity tests
  int values() const { return g == 0 ? ng : g * ng; }  // per lane
  int capacity() const { return 64 * values() * w; }
};

// Largest k that the lists of a workgroup of w wavefronts take (rtopk_filter.hpp).
constexpr int filter_max_k(int w) { return w == 4 ? 256 : 512; }
// The same for the longer lists of exact mode and the precision-bounded one.
constexpr int big_filter_max_k(int w) { return w == 4 ? 512 : 1024; }
// Candidates that either hold.
constexpr int kBigRoom = 1792;
constexpr int list_room(int w) { return w == 4 ? 512 : 1024; }
constexpr int big_list_room(int w) { return w == 4 ? 1024 : kBigRoom; }

inline bool is_aligned(uintptr_t p, uintptr_t a) { return p % a == 0; }

// Smallest listed ng with 64 * g * ng >= M.
inline int pick_ng_g4(int M) {
#define X(n) if (M <= 256 * n) return n;
  RTOPK_NG_LIST_G4(X)
#undef X
  return 32;
}
inline int pick_ng_h8(int M) {
#define X(n) if (M <= 512 * n) return n;
  RTOPK_NG_LIST_H8(X)
#undef X
  return 16;
}
// Wavefronts per row of the workgroup-per-row kernel: a lane holds up to 64 values.
inline int block_waves(int M) { return M <= 16384 ? 4 : (M <= 32768 ? 8 : 16); }

// The layout of rows of M columns.  dtype: their element type.  Requires 1 <= M <= kMaxM (kMaxBlockM for 16-bit rows and the dense-output form).
inline Shape kernel_layout(int M, int dtype) {
  Shape s{};
  s.w = 1;
  if (M > kMaxBlockM) {
    // streamed: nothing is held, so the "layout" is only the load width (full is never claimed)
    s.family = kFamStream;
    s.g = 4;
    s.w = 16;
    return s;
  }
  if (M > kMaxWaveM) {
    s.family = kFamBlock;
    s.w = block_waves(M);
    s.g = dtype == kF32 ? 4 : 8;
    // 48 or 64 values per lane: a lane's empty quarter costs as much in every pass over its values as a full one, and registers that another
    // workgroup of the compute unit could use (64 -> 48 values, us: 2000 x 20000, k = 30 precision 1e-4 40.6 -> 30.5, the k smallest 37.0 -> 28.7,
    // bfloat16 31.6 -> 23.2, dense 61.8 -> 58.5; 1000 x 9000, k = 100 13.7 -> 12.7, 12.1 -> 11.1, 10.2 -> 9.2, 15.4 -> 13.4; dense 22 x 40504, k = 56
    // 14.7 -> 12.5; nowhere slower).
    s.ng = (M <= 64 * s.w * 48 ? 48 : 64) / s.g;
  } else if (M > 512) {
    s.family = dtype == kF32 ? kFamG4 : kFamH16;
    s.g = dtype == kF32 ? 4 : 8;
    s.ng = dtype == kF32 ? pick_ng_g4(M) : pick_ng_h8(M);
  } else {
    // exactly as many values per lane as the row needs
    const int E = (M + 63) / 64;
    s.family = dtype == kF32 ? kFamSmall : kFamH16;
    if (E == 1 || E == 2) {
      s.g = E;
      s.ng = 1;
    } else if (E == 4 || E == 8) {
      s.g = dtype != kF32 && E == 8 ? 8 : 4;
      s.ng = E / s.g;
      if (dtype == kF32) s.family = kFamG4;
    } else {
      s.g = 0;
      s.ng = E;
    }
  }
  s.full = s.g != 0 && M == s.capacity();
  return s;
}

// Most rows of M columns (1537 .. 8192) that take a workgroup of four wavefronts each instead of one wavefront.  A
// wavefront alone on its SIMD walks its 32 to 128 values in series, and 128 values per lane leave room for three wavefronts on a SIMD,
// however many rows there are; the workgroup meets at half a dozen barriers instead.  Kernel times, one wavefront -> four
// (fp32, exact mode unless said otherwise, us):
//   8192 columns, k = 64: 16 rows 7.3 -> 5.5, 1024 12.5 -> 10.6, 8192 47.7 -> 45.1, 16384 90.7 -> 88.8, 32768 178 -> 180; k = 250: 16 10.8 ->
//     6.9, 8192 55.3 -> 51.2; early stopping 8192 rows 47.6 -> 45.6; dense 1024 15.3 -> 11.6, 8192 97.6 -> 89.4, 32768 381 -> 358; bfloat16
//     1024 10.2 -> 8.7, 4096 18.7 -> 17.7, 8192 29.0 -> 29.5, with early stopping 4096 18.3 -> 18.2;
//   6000: 256 8.2 -> 6.6, 2048 14.4 -> 13.2, 4096 21.7 -> 21.1 (5000 19.3 -> 19.3); early stopping 512 8.4 -> 8.1, eps 9.7 -> 9.7;
//     dense 1024 11.6 -> 10.4, 2048 17.5 -> 20.7; bfloat16 1024 9.0 -> 8.4, 2048 11.1 -> 11.1;
//   4096: 16 5.9 -> 5.1, 1024 9.1 -> 8.1, 2048 11.5 -> 11.0, 4096 15.6 -> 17.1; k = 250 2048 15.5 -> 13.1; 3000: 1024 8.0 -> 7.6, 2048 10.2 -> 10.3;
//     dense 1024 9.5 -> 8.5; bfloat16 512 6.9 -> 6.4, 1024 (3000 columns) 7.2 -> 7.3; early stopping 512 7.2 -> 7.1, eps 8.0 -> 8.4;
//   2048: k = 140 512 7.7 -> 6.2, 2048 10.1 -> 10.1; k = 64 512 6.6 -> 6.5; 1536: k = 64 512 6.1 -> 6.3.
inline int64_t workgroup_rows(int M, int k, bool half, int mode, bool dense) {
  if (M > 6144) return half ? (mode == kExact ? 6144 : 4096) : (dense ? 0x7fffffff : 24576);
  if (M > 4096) return dense ? 1024 : (mode == kExact ? (half ? 1024 : 3072) : 512);
  if (M > 2048) return mode != kExact ? 0 : (half ? 512 : (dense ? 1024 : M / 2));
  return M > 1536 && k >= 100 && mode == kExact && !half && !dense ? 1024 : 0;
}
// The layout of a call of N rows: kernel_layout(), but for these (how the workgroup then searches: block_search).
inline Shape layout_of_call(int64_t N, int M, int k, int dtype, int mode, int max_iter, bool dense) {
  Shape s = kernel_layout(M, dtype);
  if (M <= kMaxWaveM && k <= 256 && k < M && (mode != kEarly || max_iter >= 5) &&
      N <= workgroup_rows(M, k, dtype != kF32, mode, dense)) {
    s.family = kFamBlock;
    s.w = 4;
    s.g = dtype == kF32 ? 4 : 8;
    s.ng = (M <= 4096 ? 16 : 32) / s.g;
    s.full = M == s.capacity();
  }
  // Exact mode with larger k (one wavefront per row, or four wavefronts that hold 64 values per lane, -> these; us): fp32, 512 rows of 4096
  // columns, k = 300 11.4 -> 8.2, k = 512 11.0 -> 10.9, 8192 rows 36 -> 57; 4100 columns, k = 500 11.2 -> 9.8; 8192 columns, k = 300 512 rows
  // 14.3 -> 9.7, 4096 rows 36.1 -> 35.9; k = 600 in eight wavefronts 17.5 -> 12.2, 1000 15.4 -> 15.7; 16384, k = 600 17.4 -> 15.4.  bfloat16: 4096
  // columns, k = 300 512 rows 15.8 -> 8.2, 8192 rows 47 -> 55; 8192 columns, k = 512 4096 rows 53 -> 45, 16384 rows 149 -> 156; 512 rows, k = 600
  // 22.2 -> 11.9, 1000 22.5 -> 11.9, 4096 rows, k = 600 53 -> 73; 6000 columns, k = 1000 18.4 -> 11.9.
  const bool half = dtype != kF32;
  if (mode == kExact && !dense && M > 2048 && M <= 16384 && k > filter_max_k(4) && k < M) {
    const bool four = k <= big_filter_max_k(4) && M <= kMaxWaveM && N <= (half ? (M > 6144 ? 4096 : 1024) : 512);
    const bool eight = k > big_filter_max_k(4) && N <= 512 &&
                       (M <= kMaxWaveM ? (half ? M > 4096 && k <= big_filter_max_k(8) : M > 7168 && k <= 700)
                                       : k <= 700 && (half || M > 14336));
    if (four || eight) {
      s.family = kFamBlock;
      s.w = four ? 4 : 8;
      s.g = half ? 8 : 4;
      s.ng = (M <= 1024 * s.w ? 16 : 32) / s.g;
      s.full = M == s.capacity();
    }
  }
  return s;
}

// How a workgroup searches its row (rtopk_block_kernel.hpp, rtopk_filter.hpp): over the whole row, on the lists, on exact mode's
// longer lists.  Bits, for block_kernels().
enum BlockSearch : int { kSearchRow = 1, kSearchLists = 2, kSearchLongLists = 4 };

// A row's loads of g columns, and those of the wavefronts before `wave` of its w (load i is lane i % 64 of wavefront i / 64 % w).
constexpr int loads_of_row(int M, int g) { return (M + g - 1) / g; }
constexpr int loads_before(int M, int g, int w, int wave) {
  const uint32_t all = (uint32_t)loads_of_row(M, g), round = 64u * (uint32_t)w, rest = all % round, part = 64u * (uint32_t)wave;
  return (int)(all / round * part + (rest < part ? rest : part));
}

// Of the k + 1 group maxima at or above a row's floor (rtopk_filter.hpp), those that a wavefront has to have: by its share of
// the row's columns.  In equal parts, the wavefronts that a row leaves half empty find theirs far down, and as the row's floor is
// the lowest of the wavefronts', the lists overflow: normal bfloat16 rows of 3500 columns, k = 437, four wavefronts, had 1710
// candidates above it, by shares 671; 7600 columns, k = 800, eight wavefronts, 2796 and 1215 (512 rows: 16.0 -> 13.9 us; 256
// fp32 rows of 20001 columns, k = 500, 15.3 -> 12.1).  floor_shares, from the host: k + 1 maxima per load of the row, in 2^-20.
// The shares are differences of the rounded sums up to each wavefront, so that together they are k + 1 and no more (each one
// rounded up, the lists of 7 rows of 665649 columns, k = 23, whose segments leave a wavefront partly empty, overflowed now and then: 12.7
// -> 13.4 us); the sums' rounding makes up for what floor_shares has cut off.
inline uint32_t floor_shares(int M, int k, int g) { return (uint32_t)(((uint64_t)(k + 1) << 20) / (uint32_t)loads_of_row(M, g)); }
constexpr int floor_share(int M, int g, int w, int wave, uint32_t shares) {
  constexpr uint32_t up = (1u << 20) - (1u << 10);
  const uint32_t upto = ((uint32_t)loads_before(M, g, w, wave + 1) * shares + up) >> 20;
  const uint32_t share = upto - (((uint32_t)loads_before(M, g, w, wave) * shares + up) >> 20);
  return share > 0 ? (int)share : 1;
}

// Group maxima for the floor per lane of E values: of 16 values, or of a quarter of the fewer values of a lane; twice as many for
// the longer lists.
constexpr int floor_groups(int E, bool longer) { return longer && E >= 32 ? E / 8 : (E >= 48 ? E / 16 : 4); }

// Whether the lists hold ordinary rows of M columns in w wavefronts of E values per lane: with fewer group maxima than twice k
// (5/3 k for the longer lists, which have more room to spare) the floor has too many candidates, more than any list of a few
// rows in a hundred (100 normal rows each: 1600 columns, k = 220, 486 of 512 candidates at most, 256 22 % of the rows do not fit; 5000
// columns, k = 400, 1000 of 1024, 500 53 %; 4100 columns in eight wavefronts, k = 690, 1461 of 1792, 770 17 %).  What the lists
// do not hold is searched over the whole row behind them, so from there on better at once, whatever its values (16 / 512 rows, with
// lists -> without: fp32 4100 columns, k = 500 10.3 / 12.6 -> 7.9 / 9.8; bfloat16 6000 columns, k = 1000 11.0 / 15.7 -> 8.6 / 11.9).
// Lists of more than 1200 candidates, where they hold, are no better than that either (7600 columns, k = 1000, 13.5 / 16.7 -> 8.8 / 12.0;
// heavy tails 6000, k = 750 16.3 / 18.5 -> 9.7 / 13.3).
// Below the lines the search over the row is as fast on normal rows (4096 columns, k = 256, 6.7 / 7.8 with lists, 6.5 / 8.4 without;
// 512 9.4 / 10.9 and 6.8 / 8.4) but not on rows with masked entries (8.7 / 10.4 and 15.6 / 18.9; 11.4 / 12.9 and 15.7 / 18.5).
inline bool lists_hold(int M, int k, int w, int E, bool longer) {
  const int group = E / floor_groups(E, longer);
  if (longer && w == 8 && E == 16) return 20 * k * group <= 9 * M && k <= 800;
  if (longer) return 5 * k * group <= 3 * M;
  return 2 * k * group <= M;
}

// The search of a call whose layout s is a workgroup's.  N, eps_rel: what the precision-bounded mode goes by besides.
inline int block_search(const Shape& s, int M, int k, int dtype, int mode, int max_iter, bool dense, int64_t N, float eps_rel) {
  const int E = s.values();
  // Algorithm 2 with few steps ends on a threshold far below the k-th key, which the lists do not reach: the search
  // is then wasted, and with 16 wavefronts the row is read again (50000 columns, k = 256, four steps: 134 us
  // against 88 us; 32768 columns 56.6 against 56.1).  From eight (five) steps on the lists win as in exact mode.
  if (k <= filter_max_k(s.w) && (mode != kEarly || max_iter >= (s.w == 16 ? 8 : 5)))
    return lists_hold(M, k, s.w, E, false) ? kSearchLists : kSearchRow;
  if (dense || mode == kEarly || k > big_filter_max_k(s.w)) return kSearchRow;
  // The precision-bounded mode's steps follow from the k-th key and the next (steps_by_rank), and a search over the row that ends without
  // a count of k ranks its band by one lane mask after another (us, over the row -> lists: 103 x 9312, k = 360, 1e-2 15.5 -> 13.0, 1e-4 16.4 ->
  // 13.4, 1e-6 11.8 -> 12.5; 2000 x 9000, k = 300 48 -> 31, 39 -> 30, 33 -> 29; 64 x 30000, k = 750 20.3 -> 18.6, 20.8 -> 18.4, 15.8 -> 17.1; 200
  // x 25000, k = 520, 1e-6 17.7 -> 16.0).
  if (mode == kEps && (E < 48 || (N < 200 && eps_rel < 1e-5f))) return kSearchRow;
  if (E < 48) return lists_hold(M, k, s.w, E, true) ? kSearchLongLists : kSearchRow;
  // Longer lists where k is a small part of the row (us, search over the row -> lists): 12288 columns, k = 500 39 -> 36;
  // 16384, k = 400 38.5 -> 31.2; 24000, k = 600 43.4 -> 40.4, 1000 45.9 -> 50.0; 32768, k = 600 44 -> 34; 50000, k = 1000
  // 69 -> 67; 65536 188 -> 157.  16-bit rows, whose search over the row costs as much as that of fp32 rows, win throughout:
  // 16384, k = 400 48 -> 25; 24000, k = 1000 73 -> 62; 32768 53 -> 35; 50000, k = 600 83 -> 43.  Rows of whole numbers gain
  // 1.2 to 1.9 times, of heavy tails up to 1.5; sorted rows, whose lists overflow, lose 10 to 35 %.
  return (dtype != kF32 || s.w == 4 ? 24 : 40) * k <= M ? kSearchLongLists : kSearchRow;
}

// The searches that layout_of_call and block_search can ask of a workgroup layout of E values per lane in w wavefronts: those
// that are compiled.  (Layouts of fewer than 48 values per lane are for few rows only: lists with k <= 256, exact mode with more.)
constexpr int block_kernels(int E, int w, int mode, bool dense, bool half) {
  if (E >= 48) return kSearchRow | kSearchLists | (mode != kEarly && !dense ? kSearchLongLists : 0);
  if (w == 8) return mode != kExact || dense ? 0 : (half ? kSearchRow | kSearchLongLists : kSearchLongLists);
  if (mode == kExact && !dense) return kSearchRow | kSearchLists | kSearchLongLists;
  return E == 32 || dense ? (E == 16 && mode != kExact ? 0 : kSearchLists) : 0;
}

// True when (g, ng, w) is a layout of its family's lists above.  dense: in the dense-output form.
inline bool instantiated(const Shape& s, int dtype, bool dense) {
  bool small = false, g4 = false, h8 = false;
#define X(G, NG) small = small || (s.g == G && s.ng == NG);
  RTOPK_LAYOUT_LIST_SMALL(X)
#undef X
#define X(n) g4 = g4 || (s.g == 4 && s.ng == n);
  RTOPK_NG_LIST_G4(X)
#undef X
#define X(n) h8 = h8 || (s.g == 8 && s.ng == n);
  RTOPK_NG_LIST_H8(X)
#undef X
  switch (s.family) {
    case kFamSmall:
      return dtype == kF32 && s.w == 1 && small;
    case kFamG4:
      return dtype == kF32 && s.w == 1 && g4;
    case kFamH16:
      return dtype != kF32 && !dense && s.w == 1 && (small || h8 || (s.g == 4 && s.ng == 1));
    case kFamBlock:
      if (s.w != 4 && s.w != 8 && s.w != 16) return false;
      if (dtype != kF32 && dense) return false;
      return s.g == (dtype == kF32 ? 4 : 8) && (s.values() >= 48 ? s.values() == 48 || s.values() == 64 : s.w <= 8 && (s.values() == 16 || s.values() == 32));
    case kFamStream:
      return dtype == kF32 && !dense && s.w == 16 && s.g == 4;
    default:
      return false;
  }
}

// ---- rows spread over several workgroups ---------------------------------------------------------
// (rtopk_split_kernel.hpp)
// Candidates that a segment's lists hold: with nothing to search there, more than the lists of a whole row.
constexpr int segment_room(int w) { return w == 4 ? 768 : 1536; }
constexpr int kMergeRegs = 16;                // candidates per lane of a merging wavefront
constexpr int kMergeMost = 16 * 64 * kMergeRegs;  // candidates that 16 merging wavefronts hold
constexpr int kSegmentLeast = 1 + 6 + 16;     // expected of a segment at k = 1, see split_of
constexpr int kMaxSegments = kMergeMost / kSegmentLeast;
constexpr int kSegmentHeadBytes = 16;
constexpr int64_t kSplitScratch = 128ll << 20;

// How a call is split: `segments` per row of `length` columns (the last may be shorter), lists of up to `cap` candidates,
// workgroups of w wavefronts with ng groups per lane, merge_waves wavefronts per row to merge.  segments = 0: not at all.
struct Split {
  int segments, length, cap, w, ng, merge_waves;
  bool big;  // lists of up to kBigRoom candidates, floors from eight groups per lane
  int64_t rows;  // rows per pair of launches, so that the scratch memory stays bounded
  int64_t bytes() const { return rows * segments * (kSegmentHeadBytes + (int64_t)cap * 8); }
};

// Algorithm 2 with fewer than eight steps usually ends on a threshold far below the lists' floor.  The lists still decide every
// step (a count at or below the floor is more than k), and the merging workgroup writes the row's first k keys from the row itself, which
// costs it a pass up to the k-th of them.  A row that one workgroup holds in registers needs no such pass and stays there (512 x 50000,
// k = 100, four steps 32 us, split 39); a streamed one is read twice by one workgroup in any case (us, streamed -> split: 1 x 131072, k = 50
// four steps 39 -> 9.6; 64 x 262144, k = 600 three 126 -> 30; 1 x 10^6, k = 300 208 -> 19; 1024 x 131072 two 214 -> 116, six 119 -> 104; masked rows
// 200 -> 31, sorted ones 228 -> 81).  Enough rows of 2^19 columns and more to stream at the full rate lose 3 to 7 % with one step, or with five and
// more (512 x 524288, one 188 -> 194, four 331 -> 188, six 184 -> 192; 256 x 10^6, six 178 -> 192).
inline bool splits_early(int64_t N, int M, int max_iter) {
  if (max_iter >= 8) return true;
  if (max_iter < 1 || M <= kMaxBlockM) return false;
  return (max_iter >= 2 && max_iter <= 4) || M < 1 << 19 || N * M < 1ll << 28;
}
// Columns of each of `segments` segments, and the values per lane of w wavefronts that hold them.
constexpr int segment_length(int M, int segments) { return ((M + segments - 1) / segments + 3) & ~3; }
constexpr int segment_values(int length, int w) { return length <= w * 3072 ? 48 : 64; }
// Segments of 16384 columns where those of 32768, `wide` of them in all, give every compute unit two workgroups or more: of the smaller workgroups five
// share a compute unit instead of two, but the merge has twice the candidates; where a merge of four wavefronts holds these, up to four workgroups for
// each compute unit, eight with up to eight lists to a row.  Early stopping with few steps: the shorter segments' floors lie lower, so that fewer rows
// end below them and are walked again.  Otherwise it pays the less, the fuller the lanes of the longer segments are (to 27/32, to 31/32, beyond, full),
// the more values they hold in the shorter ones (48 -> 64) and the larger k is; the more, where rows start off 16-byte boundaries.  Time with
// 32768-column segments over time with 16384-column ones, at 520, 860, 1400 and 2040 longer segments in all (exact mode; eight and sixteen steps and
// precisions differ from it by 0.02):
//   lanes to 27/32: 50000, k = 48 1.14 1.13 1.10 1.06, 134 1.12 1.12 1.07 1.02, 200 1.02 1.02 0.99 0.96, 80000, k = 200 1.11 1.06 1.02 0.99, 80001 1.11
//     1.06 1.01 0.99; to 31/32: 62000, k = 48 1.10 1.09 1.05 1.01, 110 1.11 1.08 1.04 0.98, 134 1.10 1.07 1.02 0.99, 200 1.01 0.99 0.98 0.93, 59999, k = 110
//     1.12 1.10 1.05 1.01, 160 1.06 1.06 1.03 0.97, 94000, k = 48 1.10 1.12 1.09 1.05; beyond: 128000, k = 48 1.12 1.06 1.01 0.94, 127999 1.11 1.08 1.03
//     0.97; full: 65536, 98304, 131072, k = 48 1.08 0.97 0.91 0.89, k = 160 1.02 0.94 0.87 0.87, 65535, k = 48 1.11 1.02 0.93 0.90, 160 1.05 1.01 0.91 0.88;
//   three short segments: 34424, k = 160 1.10 1.05 1.06 1.04, 250 1.02 0.97 0.98 0.96, with 64 values 41000, k = 134 1.05 1.01 1.04 1.03, 160 1.05 1.01 1.01
//     1.02, 250 0.96 0.94 0.94 0.94; five with 64 values: 70000, k = 48 1.06 1.01 0.99 0.98, 200 1.00 0.98 0.96 0.93, 67571, k = 48 1.04 1.04 1.03 1.03;
//   four steps: 112484, k = 134 1.45 1.33 1.16 1.11, 98304, k = 134 1.35 1.12 1.01 1.03, 70000, k = 8 1.06 0.95 1.00 0.96.
inline bool shorter_segments(int M, int k, int mode, int max_iter, int64_t wide, int64_t candidates) {
  const int short_ones = (M + 16383) / 16384, length = segment_length(M, (M + 32767) / 32768), values = segment_values(length, 8);
  const int lanes = 512 * values, most = short_ones > 8 ? 4 * 256 : 8 * 256;
  const bool more_values = segment_values(segment_length(M, short_ones), 4) > values, off = M % 4 != 0;
  int line = most;
  if (mode == kEarly && max_iter <= 5) {
  } else if (1000 * length >= 997 * lanes) {
    line = off && k <= 112 ? 860 : (k <= 160 ? 640 : 0);
  } else if (short_ones == 3) {
    line = k <= (more_values ? 160 : 200) ? most : 0;
  } else if (more_values) {
    line = off && k <= 112 ? most : (k <= 160 ? 560 : 0);
  } else if (32 * length < 27 * lanes) {
    line = k <= 96 ? most : (k <= 160 ? 1664 : (off ? 1280 : 640));
  } else {
    line = k <= (off ? 112 : 56) ? most : (k <= (off ? 160 : 112) ? 1536 : (k <= 160 ? 1280 : (k <= 200 ? 640 : 0)));
    if (32 * length >= 31 * lanes) line = line < (off ? 1408 : 1280) ? line : (off ? 1408 : 1280);
  }
  return wide < (line < most ? line : most) && candidates <= 4 * 64 * kMergeRegs;
}
// wide_only: segments of 32768 columns whatever the number of rows.
inline Split split_of(int64_t N, int M, int k, int mode, int max_iter, bool wide_only = false) {
  Split s{};
  // Up to 32768 columns one workgroup per row does as well.
  if (M <= 32768 || N < 1 || k > filter_max_k(8) || (mode == kEarly && !splits_early(N, M, max_iter))) return s;
  // A segment's candidates: 1.2 to 1.35 k, and the spread of its wavefronts' floors, which weighs when k is small: `usual` is
  // seldom exceeded on ordinary rows (k = 64: 176 at most, k = 512: 1012 in one segment of 200).  The merging workgroup's
  // registers hold what its row can have, unless that is beyond 16 wavefronts: there they hold what is expected of the row.
  int root = 1;
  while (root * root < k) ++root;
  const int usual = k + k / 3 + 10 * root + 24, expected = k + k / 3 + 6 * root + 16;
  // Segments of 32768 columns, unless those would not give every compute unit two workgroups and those of 16384, which have
  // twice the candidates in all, still fit the merge; or, up to twice that many rows and more, where shorter_segments says so.
  s.w = 8;
  const int64_t wide = N * ((M + 32767) / 32768), narrow = (M + 16383) / 16384;
  if (!wide_only && k <= filter_max_k(4) && (wide < 2 * 256 ? narrow * expected <= kMergeMost : shorter_segments(M, k, mode, max_iter, wide, narrow * usual))) s.w = 4;
  const int most = s.w * 4096;
  s.segments = (M + most - 1) / most;
  if ((int64_t)s.segments * expected > kMergeMost) {
    s.segments = 0;
    return s;
  }
  s.length = segment_length(M, s.segments);
  s.ng = segment_values(s.length, s.w) / 4;
  const int64_t need = (int64_t)s.segments * usual, per_wave = 64 * kMergeRegs;
  s.merge_waves = need <= 4 * per_wave ? 4 : (need <= 8 * per_wave ? 8 : 16);
  const int share = (int)(s.merge_waves * per_wave / s.segments);
  s.cap = share > usual ? share : usual;
  if (s.cap > 4 * k + 640) s.cap = 4 * k + 640;
  if (s.cap > segment_room(s.w)) s.cap = segment_room(s.w);
  if (mode == kEarly && max_iter < 8) s.merge_waves = 16;  // for the pass over the row
  const int64_t per_row = s.segments * (kSegmentHeadBytes + (int64_t)s.cap * 8);
  s.rows = kSplitScratch / per_row;
  if (s.rows < 1) s.rows = 1;
  if (s.rows > N) s.rows = N;
  return s;
}

// Rows of more than kMaxBlockM columns that split_of leaves to one streaming workgroup, because k is above its lists' limit or
// their candidates would not fit the merge: lists of up to kBigRoom candidates, from segments of 32768 columns, or of 65536
// where the merge would not hold twice as many lists; 40 candidates per merging lane where 16 would not do.  (16 rows of
// 131072 columns, k = 600: streamed 46.6 us, split 15.9; 16 rows of 2^20, k = 800: 165 -> 50; 1000 rows of 131072, k = 700:
// 151 -> 121.)  The floors come from eight groups of eight values per lane here, so a list has 1.1 to 1.35 k candidates at
// k = 512 .. 1024.  Lists of 16 wavefronts, whose floors spread more, are expected to hold 1.5 k.
constexpr int kBigMaxK = 1024;
constexpr int kMergeRegsBig = 40;  // candidates per lane that 16 merging wavefronts hold at most
inline Split split_big_of(int64_t N, int M, int k, int mode, int max_iter) {
  Split s{};
  if (M <= kMaxBlockM || N < 1 || k > kBigMaxK || (mode == kEarly && !splits_early(N, M, max_iter))) return s;
  int root = 1;
  while (root * root < k) ++root;
  s.big = true;
  s.ng = 16;
  s.merge_waves = 16;
  int most = kMergeMost;
  for (int round = 0; round < 3; ++round) {
    s.w = round == 0 ? 8 : 16;
    if (round == 2) most = 16 * 64 * kMergeRegsBig;
    s.segments = (M + s.w * 4096 - 1) / (s.w * 4096);
    if ((int64_t)s.segments * (k + (s.w == 8 ? k / 3 : k / 2) + 6 * root + 16) <= most) break;
    s.segments = 0;
  }
  if (s.segments < 2) return Split{};
  s.length = ((M + s.segments - 1) / s.segments + 3) & ~3;
  s.cap = most / s.segments < kBigRoom ? most / s.segments : kBigRoom;  // no row has more than the merge holds
  s.rows = kSplitScratch / (s.segments * (kSegmentHeadBytes + (int64_t)s.cap * 8));
  if (s.rows < 1) s.rows = 1;
  if (s.rows > N) s.rows = N;
  return s;
}

// The split of a call that is lent `lent` bytes of scratch memory.  Segments of 16384 columns take nearly twice as much as those of 32768, which are
// what more rows take: memory that serves a batch serves every smaller one, with the longer segments where the shorter ones do not fit (2048 x 50000, k =
// 100: one workgroup per row, without memory, 135 us, 32768-column segments 79).
inline Split split_for(int64_t N, int M, int k, int mode, int max_iter, int64_t lent = INT64_MAX) {
  Split s = split_of(N, M, k, mode, max_iter);
  if (s.segments > 0 && s.bytes() > lent) s = split_of(N, M, k, mode, max_iter, true);
  if (s.segments == 0) s = split_big_of(N, M, k, mode, max_iter);
  return s.segments > 0 && s.bytes() <= lent ? s : Split{};
}

// Largest max_iter that is evaluated literally.  Each step of Algorithm 2 halves hi - lo, so on finite
// fp32 input the rounded midpoint equals lo or hi after at most ~300 steps (from a range of 2^129 down
// to the smallest subnormal, plus 24 mantissa bits); from then on a step changes neither bound, so a
// larger step count gives bit-identical output.  The clamp keeps a huge max_iter (a caller's way of
// saying "no early stop") from spinning on rows whose k-th place is tied and so never count exactly k.
constexpr int kMaxIterClamp = 512;

// True when the byte ranges [a, a + na) and [b, b + nb) share a byte.
inline bool ranges_overlap(uintptr_t a, uint64_t na, uintptr_t b, uint64_t nb) {
  if (na == 0 || nb == 0) return false;
  return a < b + nb && b < a + na;
}

}  // namespace rtopk
