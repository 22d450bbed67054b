// CPU-only sanitizer target (built and run by tests/test_sanitize_cpu.py with
// -fsanitize=address,undefined): the oracle, the input generator and the library's host-side
// choice of layouts and splits, exercised in one process so that any out-of-bounds access, use of an uninitialised
// index, signed overflow or misaligned access in them aborts the test.
//
//   1. the Algorithm 2 hand traces of tests/golden/alg2_handtrace.txt against the sanitized oracle;
//   2. brute force (a stable sort written out here) against the oracle's exact mode, Algorithm 1 at
//      epsilon = 0 and the k-smallest variant on tiny tie-heavy rows from the sanitized generator;
//   3. the layout that is launched for every row width 1..65536 (and a sample of the streamed widths up to
//      2^24), every element type and the dense form: it must be compiled, hold the row and
//      be no wider than its kernels take for granted;
//   4. how rows are spread over several workgroups, over widths, k, row counts, modes and steps: segments, lists and
//      scratch memory within what the kernels and the merge hold, and what is lent for a batch enough for smaller ones.
//
// Usage: sanitize_main <path to alg2_handtrace.txt>.  Exit code 0 = all checks passed.
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>

#include "rtopk_shape.hpp"

extern "C" {
int oracle_topk_exact(const float* in, int64_t N, int32_t M, int32_t k, float* out_vals, int32_t* out_idx);
int oracle_topk_earlystop(const float* in, int64_t N, int32_t M, int32_t k, int32_t max_iter, float* out_vals,
                          int32_t* out_idx);
int oracle_alg1(const float* in, int64_t N, int32_t M, int32_t k, float eps_rel, int32_t collect, float* out_vals,
                int32_t* out_idx, int32_t* out_iters);
int oracle_topk_exact_smallest(const float* in, int64_t N, int32_t M, int32_t k, float* out_vals, int32_t* out_idx);
int oracle_maxk_backward(const float* grad_vals, const int32_t* idx, int64_t N, int32_t M, int32_t k, float* grad_in);
int wl_fill_normal_ties(float* out, int64_t N, int32_t M, uint64_t seed, double p, int32_t levels, double level0,
                        double step);
int wl_fill_normal(float* out, int64_t N, int32_t M, uint64_t seed, int32_t row_scale, double scale_lo,
                   double scale_hi);
}

static int g_failures = 0;
#define CHECK(cond, ...)                          \
  do {                                            \
    if (!(cond)) {                                \
      std::fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
      std::fprintf(stderr, __VA_ARGS__);          \
      std::fprintf(stderr, "\n");                 \
      if (++g_failures > 20) std::exit(1);        \
    }                                             \
  } while (0)

// ---- 1. hand traces -------------------------------------------------------------------------------
static int run_hand_traces(const char* path) {
  std::ifstream f(path);
  if (!f) {
    std::fprintf(stderr, "cannot open %s\n", path);
    return -1;
  }
  std::string line;
  int cases = 0;
  while (std::getline(f, line)) {
    if (line.empty() || line[0] == '#') continue;
    std::vector<std::string> part;
    std::stringstream ss(line);
    std::string item;
    while (std::getline(ss, item, '|')) part.push_back(item);
    CHECK(part.size() == 4, "malformed line: %s", line.c_str());
    if (part.size() != 4) continue;
    std::vector<float> v;
    {
      std::stringstream s0(part[0]);
      float x;
      while (s0 >> x) v.push_back(x);
    }
    const int k = std::atoi(part[1].c_str()), mi = std::atoi(part[2].c_str());
    std::vector<int32_t> want;
    {
      std::stringstream s3(part[3]);
      int x;
      while (s3 >> x) want.push_back(x);
    }
    CHECK((int)want.size() == k, "k does not match the expected columns: %s", line.c_str());
    std::vector<float> ov((size_t)k);
    std::vector<int32_t> oi((size_t)k);
    const int rc = oracle_topk_earlystop(v.data(), 1, (int32_t)v.size(), k, mi, ov.data(), oi.data());
    CHECK(rc == 0, "oracle_topk_earlystop rc %d", rc);
    CHECK(oi == want, "hand trace differs: %s", line.c_str());
    for (int j = 0; j < k; ++j) CHECK(ov[(size_t)j] == v[(size_t)oi[(size_t)j]], "value is not a copy of the input");
    ++cases;
  }
  return cases;
}

// ---- 2. brute force ---------------------------------------------------------------------------------
// The plain definition: order columns by value descending (ascending for the k smallest), ties by column
// ascending; take the first k; report them in ascending column order.
static std::vector<int32_t> brute(const float* v, int M, int k, bool smallest) {
  std::vector<int32_t> order((size_t)M);
  for (int i = 0; i < M; ++i) order[(size_t)i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
    return smallest ? v[a] < v[b] : v[a] > v[b];
  });
  order.resize((size_t)k);
  std::sort(order.begin(), order.end());
  return order;
}

static int run_brute_force() {
  int rows_checked = 0;
  for (int M : {1, 2, 3, 5, 8, 12, 17, 33}) {
    const int N = 200;
    std::vector<float> x((size_t)N * M);
    // half of the entries snapped to three shared levels: ties within every row
    CHECK(wl_fill_normal_ties(x.data(), N, M, 900 + (uint64_t)M, 0.5, 3, -0.5, 0.5) == 0, "generator failed");
    for (int i = 0; i < N * M; i += 7) x[(size_t)i] = (i % 14 == 0) ? -0.0f : 0.0f;  // signed zeros
    for (int k = 1; k <= M; ++k) {
      std::vector<float> ov((size_t)N * k), av((size_t)N * k), sv((size_t)N * k);
      std::vector<int32_t> oi((size_t)N * k), ai((size_t)N * k), si((size_t)N * k), it((size_t)N);
      CHECK(oracle_topk_exact(x.data(), N, M, k, ov.data(), oi.data()) == 0, "exact rc");
      CHECK(oracle_alg1(x.data(), N, M, k, 0.0f, 1, av.data(), ai.data(), it.data()) == 0, "alg1 rc");
      CHECK(oracle_topk_exact_smallest(x.data(), N, M, k, sv.data(), si.data()) == 0, "smallest rc");
      for (int r = 0; r < N; ++r) {
        const float* row = x.data() + (size_t)r * M;
        const std::vector<int32_t> want = brute(row, M, k, false), want_s = brute(row, M, k, true);
        for (int j = 0; j < k; ++j) {
          const size_t o = (size_t)r * k + j;
          CHECK(oi[o] == want[(size_t)j], "exact: M=%d k=%d row %d", M, k, r);
          CHECK(ai[o] == want[(size_t)j], "alg1 eps=0: M=%d k=%d row %d", M, k, r);
          CHECK(si[o] == want_s[(size_t)j], "smallest: M=%d k=%d row %d", M, k, r);
          CHECK(ov[o] == row[oi[o]] && av[o] == row[ai[o]] && sv[o] == row[si[o]], "values are not copies");
        }
        ++rows_checked;
      }
    }
  }
  // the backward edge: gradients scattered to the saved columns, zero elsewhere
  {
    const int N = 50, M = 37, k = 9;
    std::vector<float> x((size_t)N * M), g((size_t)N * k), v((size_t)N * k), gin((size_t)N * M);
    std::vector<int32_t> idx((size_t)N * k);
    CHECK(wl_fill_normal(x.data(), N, M, 77, 0, 0, 0) == 0 && wl_fill_normal(g.data(), N, k, 78, 0, 0, 0) == 0, "generator");
    CHECK(oracle_topk_exact(x.data(), N, M, k, v.data(), idx.data()) == 0, "exact rc");
    CHECK(oracle_maxk_backward(g.data(), idx.data(), N, M, k, gin.data()) == 0, "backward rc");
    for (int r = 0; r < N; ++r) {
      std::vector<float> want((size_t)M, 0.0f);
      for (int j = 0; j < k; ++j) want[(size_t)idx[(size_t)r * k + j]] = g[(size_t)r * k + j];
      for (int c = 0; c < M; ++c) CHECK(gin[(size_t)r * M + c] == want[(size_t)c], "backward scatter row %d col %d", r, c);
    }
  }
  return rows_checked;
}

// ---- 3. the layouts that are launched --------------------------------------------------------------
static long run_shape_sweep() {
  long n = 0;
  for (int M = 1; M <= rtopk::kMaxBlockM; ++M) {
    for (int dtype : {rtopk::kF32, rtopk::kF16, rtopk::kBF16}) {
      for (int dense = 0; dense <= (dtype == rtopk::kF32 ? 1 : 0); ++dense) {
        const rtopk::Shape s = rtopk::kernel_layout(M, dtype);
        CHECK(rtopk::instantiated(s, dtype, dense != 0), "M=%d dtype=%d dense=%d: (%d,%d,%d) family %d not compiled",
              M, dtype, dense, s.g, s.ng, s.w, s.family);
        CHECK(s.capacity() >= M, "M=%d: layout (%d,%d,%d) holds only %d", M, s.g, s.ng, s.w, s.capacity());
        CHECK(s.full == (s.g != 0 && s.capacity() == M), "M=%d: full flag", M);
        CHECK((s.w == 1) == (M <= rtopk::kMaxWaveM), "M=%d: wavefronts per row %d", M, s.w);
        CHECK(s.w == 1 ? s.values() <= 128 : s.values() <= 64, "M=%d: %d values per lane", M, s.values());
        // the vector loads stay inside the row, and the groups that the kernels take for whole are: up to 512
        // columns the row fills all but the last value of a lane, beyond them no shorter layout of the list holds it
        CHECK(M >= (s.g == 0 ? 4 : s.g), "M=%d: narrower than a load of %d", M, s.g);
        if (M <= 512) {
          CHECK(s.values() == (M + 63) / 64, "M=%d: %d values per lane", M, s.values());
        } else if (s.w == 1) {
          rtopk::Shape less = s;
          while (--less.ng > 0 && !rtopk::instantiated(less, dtype, dense != 0)) {
          }
          CHECK(less.ng == 0 || less.capacity() < M, "M=%d: (%d,%d) would do", M, less.g, less.ng);
        } else {
          CHECK(64 * s.w * s.values() / 2 < M, "M=%d: (%d,%d,%d) is half empty", M, s.g, s.ng, s.w);
        }
        ++n;
      }
    }
  }
  // beyond the widest row a workgroup holds: fp32 rows are streamed
  for (int64_t M = rtopk::kMaxBlockM + 1; M <= rtopk::kMaxM; M += (M < 70000 ? 1 : 9973)) {
    const rtopk::Shape s = rtopk::kernel_layout((int)M, rtopk::kF32);
    CHECK(s.family == rtopk::kFamStream && rtopk::instantiated(s, rtopk::kF32, false), "M=%ld: not streamed", (long)M);
    ++n;
  }
  return n;
}

// ---- 4. rows spread over several workgroups ---------------------------------------------------------
static void check_split(const rtopk::Split& s, int64_t M, int k, int64_t N) {
  CHECK(M > 32768 && k <= 512, "M=%ld k=%d is split", (long)M, k);
  CHECK(s.segments >= 2 && s.segments <= rtopk::kMaxSegments, "M=%ld k=%d: %d segments", (long)M, k, s.segments);
  CHECK(s.w == 4 || s.w == 8, "M=%ld: %d wavefronts", (long)M, s.w);
  CHECK(k <= rtopk::filter_max_k(s.w), "M=%ld k=%d: lists of %d wavefronts", (long)M, k, s.w);
  CHECK(s.length % 4 == 0 && s.length <= 64 * s.w * 4 * s.ng && (s.ng == 12 || s.ng == 16), "M=%ld: length %d", (long)M, s.length);
  const int64_t last = M - (int64_t)(s.segments - 1) * s.length;
  CHECK(last > 0 && last <= s.length, "M=%ld: last segment of %ld", (long)M, (long)last);
  // every wavefront has group maxima (of 16 values per lane) for its share of the floor
  CHECK(last >= 64 * s.w * 4 * 4 + 64 * s.w * 4, "M=%ld: last segment of %ld in %d wavefronts", (long)M, (long)last, s.w);
  CHECK(s.cap > k && s.cap <= rtopk::segment_room(s.w), "M=%ld k=%d: lists of %d", (long)M, k, s.cap);
  CHECK(s.merge_waves == 4 || s.merge_waves == 8 || s.merge_waves == 16, "M=%ld: %d merging", (long)M, s.merge_waves);
  if (s.merge_waves < 16)
    CHECK((int64_t)s.segments * s.cap <= (int64_t)s.merge_waves * 64 * rtopk::kMergeRegs, "M=%ld k=%d: more than the merge holds", (long)M, k);
  CHECK(s.rows >= 1 && s.rows <= N && s.rows * s.segments <= 0x7fffffff, "M=%ld N=%ld: %ld rows", (long)M, (long)N, (long)s.rows);
  CHECK(s.rows == 1 || s.bytes() <= rtopk::kSplitScratch, "M=%ld N=%ld: %ld bytes", (long)M, (long)N, (long)s.bytes());
}

static long run_split_sweep() {
  const int64_t counts[] = {1, 2, 15, 16, 64, 128, 255, 256, 511, 512, 700, 1000, 1023, 1024, 2047, 2048, 100000};
  long n = 0;
  for (int64_t M = 32760; M <= rtopk::kMaxM; M += (M < 33000 || (M > 65500 && M < 65600)) ? 1 : M / 61 + 1) {
    for (int k : {1, 2, 7, 33, 64, 100, 200, 255, 256, 257, 400, 511, 512, 513, 1000}) {
      for (int mode : {(int)rtopk::kExact, (int)rtopk::kEarly, (int)rtopk::kEps}) {
        for (int steps : {8, 0, 1, 2, 4, 5, 7}) {
          if (mode != rtopk::kEarly && steps != 8) continue;
          const bool few = mode == rtopk::kEarly && steps < 8;  // (these go by the number of rows, too)
          int64_t most = -1;  // memory that serves the batches up to this one, from the largest down
          for (int c = (int)(sizeof(counts) / sizeof(counts[0])) - 1; c >= 0; --c) {
            const int64_t N = counts[c];
            const rtopk::Split s = rtopk::split_of(N, (int)M, k, mode, steps);
            ++n;
            if (s.segments == 0) {
              if (!few) CHECK(rtopk::split_of(1 << 20, (int)M, k, mode, steps).segments == 0, "M=%ld k=%d: split for many rows but not for %ld", (long)M, k, (long)N);
            } else {
              CHECK(!few || (steps >= 1 && M > rtopk::kMaxBlockM && s.merge_waves == 16), "M=%ld: %d steps, %d merging", (long)M, steps, s.merge_waves);
              check_split(s, M, k, N);
            }
            const rtopk::Split any = rtopk::split_for(N, (int)M, k, mode, steps);
            if (any.segments > 0) CHECK(rtopk::split_for(N, (int)M, k, mode, steps, any.bytes() - 1).bytes() < any.bytes(), "M=%ld k=%d N=%ld: more than was lent", (long)M, k, (long)N);
            if (most > 0) {
              const rtopk::Split with = rtopk::split_for(N, (int)M, k, mode, steps, most);
              CHECK(with.segments > 0 && with.bytes() <= most, "M=%ld k=%d: %ld rows not split with the memory of more", (long)M, k, (long)N);
              if (s.segments > 0) check_split(with, M, k, N);
            }
            if (any.segments > 0 && (most < 0 || any.bytes() < most)) most = any.bytes();
          }
        }
      }
    }
  }
  return n;
}

static void run_overlaps() {
  // range overlap helper
  CHECK(!rtopk::ranges_overlap(100, 10, 110, 10), "adjacent ranges do not overlap");
  CHECK(rtopk::ranges_overlap(100, 11, 110, 10), "one shared byte");
  CHECK(rtopk::ranges_overlap(100, 50, 120, 5), "containment");
  CHECK(!rtopk::ranges_overlap(100, 0, 100, 10), "empty range");
  CHECK(!rtopk::ranges_overlap(~(uintptr_t)0 - 7, 8, 0, 8), "top of the address space");
}

int main(int argc, char** argv) {
  if (argc < 2) {
    std::fprintf(stderr, "usage: %s <alg2_handtrace.txt>\n", argv[0]);
    return 2;
  }
  const int traces = run_hand_traces(argv[1]);
  if (traces < 0) return 2;
  const int rows = run_brute_force();
  const long shapes = run_shape_sweep(), splits = run_split_sweep();
  run_overlaps();
  std::printf("hand traces %d, brute-force rows %d, shapes %ld, splits %ld, failures %d\n", traces, rows, shapes, splits, g_failures);
  return g_failures == 0 ? 0 : 1;
}
