// Backward edge of the MaxK non-linearity for gfx950 (MI355X).
//
// RTop-K (arXiv 2409.00822) is used as the non-linearity of a MaxK-GNN layer (Section 1 / Fig. 1;
// Section 4.3 measures it inside training): forward, a row keeps its k selected entries and every other
// entry becomes zero, so the derivative with respect to the row is that same 0/1 mask.  With the k
// columns saved by the forward pass (rtopk_rowwise*: idx[N][k]) the backward step is pure data movement:
//
//   scatter:  grad_in[r][c]  = grad_vals[r][j] if c == idx[r][j] for some j, else 0      ([N][k] -> [N][M])
//   gather:   grad_vals[r][j] = grad_out[r][idx[r][j]]                                     ([N][M] -> [N][k])
//
// Both are bound by HBM bandwidth; the kernels below exist to keep every global access coalesced.
// A column outside [0, M) is ignored by the scatter and yields 0 in the gather, so a corrupt index
// cannot make either kernel touch memory outside its buffers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rtopk_kernel.hpp"

namespace rtopk {

// A wavefront of the scatter owns a chunk of the dense matrix, which may cut rows, one of the gather whole rows of it; both are contiguous, and so are
// their pairs in the [N][k] arrays.  So both kernels walk the pairs as one list, 64 neighbours to an instruction, whatever k is: BATCH instructions' worth in
// registers, as many as the wavefront has or 16, loaded together, while the chunk is cleared or the rows are loaded.  All loads are unconditional (lanes past
// the end repeat the last): behind a branch each would be waited for alone.  What bounds both is HBM, given enough loads in flight.  Measured against 2, 4, 8
// or 16 whole rows with the lanes divided among them, dword accesses where M is no multiple of four and a loop over the row for k > 64, us, matrices and
// pairs from three sets in turn: 1048576 x 251, k = 31 scatter 339 -> 203, gather 537 -> 245; x 250, k = 100 685 -> 263, 726 -> 300; x 256, k = 128 638 -> 290,
// 371 -> 285, k = 32 207 -> 207, 202 -> 201 (byte columns; int32 ones 228 -> 224, 219 -> 217); 262144 x 777, k = 40 267 -> 147, 309 -> 154; 131072 x 2048, k =
// 100 189 -> 193, 191 -> 191.

// n / d for n up to 3 * 2048 and d up to 2048, exactly: n * (by - 2^32 / d) < 2^32 / d.  by: ceil(2^32 / d), 0 where that is 2^32.
__device__ __forceinline__ int quotient(int n, uint32_t by) { return by == 0 ? n : (int)__umulhi((uint32_t)n, by); }
inline uint32_t divisor(int d) { return 0xffffffffu / (uint32_t)d + 1; }

// An element of a pair.  STREAM: with the non-temporal hint, which keeps what is read once out of the caches' way; not where wavefronts share lines,
// which are then read again from memory (the scatter with rows that a chunk cuts, inputs cold: 1048576 x 251, k = 31 243 -> 213 us without it, 131072 x
// 2048, k = 100 250 -> 220; 1048576 x 256, k = 32, where none are shared, 225 without, 219 with).
template <bool STREAM, typename T>
__device__ __forceinline__ T load_pair(const T* p) {
  return STREAM ? __builtin_nontemporal_load(p) : *p;
}

// Floats that p lies behind a boundary of n of them.
__device__ __host__ __forceinline__ int floats_behind(const float* p, int n) { return (int)((reinterpret_cast<uintptr_t>(p) >> 2) & (n - 1)); }
// out[0..n) = image[pad..pad + n), by `threads` threads of which this is number `tid`.  pad: floats that `out` lies behind a 16-byte boundary, so that
// whole quads of the image leave as aligned 128-bit stores; what precedes and follows them goes one by one.  ALIGNED: pad is 0, n a multiple of four.
template <bool ALIGNED>
__device__ __forceinline__ void store_image(float* __restrict__ out, const float* image, int n, int pad, int tid, int threads) {
  const uint4* quads = reinterpret_cast<const uint4*>(image);
  if constexpr (ALIGNED) {
    for (int q = tid; q < (n >> 2); q += threads) store_streaming(reinterpret_cast<uint4*>(out) + q, quads[q]);
  } else {
    const int q0 = pad != 0 ? 1 : 0, q1 = (pad + n) >> 2;
    for (int q = q0 + tid; q < q1; q += threads) store_streaming(reinterpret_cast<uint4*>(out - pad + 4 * q), quads[q]);
    const int head = pad != 0 ? min(4 - pad, n) : 0, tail = max(4 * q1 - pad, head);
    if (tid < head) out[tid] = image[pad + tid];
    if (tid < n - tail) out[tail + tid] = image[pad + tail + tid];
  }
}
__device__ __forceinline__ void wavefront_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- scatter, narrow rows: one wavefront per chunk of the output, which is assembled in LDS ---------------
//
// Zero fill, one 4-byte LDS write per saved column, then the image leaves back to back: HBM sees each output byte written once, in order. The
// output is cut at 128-byte boundaries, not between rows: a line that two wavefronts write parts of costs two writes (1048576 x 251, k = 31, whole
// rows per wavefront 263 us, chunks 233); of the rows that a chunk cuts both sides load the pairs and keep their own.
// packed: chunk, skew << 12, whole << 17, so that the arguments are no more than 64 bytes, a line that the host writes (with 72 bytes a call took 3.96 us
// of host time, now 3.83, and behind a selection, 79 x 235 to 7975 x 256, both 9.35, now 9.0).
template <typename IdxT, int BATCH, bool STREAM>
__global__ void __launch_bounds__(kWave)
    maxk_scatter_rows_kernel(const float* __restrict__ grad_vals, const IdxT* __restrict__ idx, float* __restrict__ grad_in, int64_t elements,
                             double per_m, int M, int k, uint32_t by, uint32_t by_m, uint32_t packed) {
  const int chunk = (int)(packed & 0xfffu), skew = (int)(packed >> 12 & 31u), whole = (int)(packed >> 17);
  extern __shared__ __attribute__((aligned(16))) float s_rows[];  // [chunk]
  const int lane = threadIdx.x;
  // The chunk's elements are [start, start + chunk) of the matrix as far as it goes; the first chunk starts `skew` before it.
  const int64_t start = (int64_t)blockIdx.x * chunk - skew;
  const int from = start < 0 ? skew : 0, to = elements - start < chunk ? (int)(elements - start) : chunk;
  const int64_t begin = start + from;
  int64_t r0;
  if (whole > 0) {  // rows that every chunk holds: none is cut (the arithmetic below comes before the first load: 2 %)
    r0 = (int64_t)blockIdx.x * whole;
  } else {
    r0 = (int64_t)((double)begin * per_m);  // begin / M, or one off
    const int64_t rem = begin - r0 * M;
    r0 += rem < 0 ? -1 : (rem >= M ? 1 : 0);
    r0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)r0 >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)r0));
  }
  const int at_row = (int)(r0 * M - start);  // where row r0 starts in the chunk, up to M - 1 before it
  const int pairs = (quotient(to - 1 - at_row, by_m) + 1) * k;
  const float* gv = grad_vals + r0 * (int64_t)k;
  const IdxT* ix = idx + r0 * (int64_t)k;
  float g[BATCH];
  int c[BATCH];
  auto load = [&](int p0) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int at = min(p0 + i * kWave + lane, pairs - 1);
      g[i] = load_pair<STREAM>(gv + at);
      c[i] = (int)load_pair<STREAM>(ix + at);
    }
  };
  load(0);
  for (int q = lane; q < chunk >> 2; q += kWave) reinterpret_cast<float4*>(s_rows)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  wavefront_lds_order();
  for (int p0 = 0;;) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) asm volatile("" : "+v"(g[i]), "+v"(c[i]));  // (or the loads move to their uses)
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int p = p0 + i * kWave + lane, at = at_row + quotient(p, by) * M + c[i];
      if (p < pairs && (unsigned)c[i] < (unsigned)M && (unsigned)at < (unsigned)chunk) s_rows[at] = g[i];
    }
    p0 += BATCH * kWave;
    if (p0 >= pairs) break;
    load(p0);
  }
  wavefront_lds_order();
  float* out = grad_in + start;
  if (to - from == chunk) {  // uniform
#pragma unroll 1
    for (int q = lane; q < chunk >> 2; q += kWave) store_streaming(reinterpret_cast<uint4*>(out) + q, reinterpret_cast<const uint4*>(s_rows)[q]);
  } else {  // the first or the last
#pragma unroll 1
    for (int j = from + lane; j < to; j += kWave) out[j] = s_rows[j];
  }
}

// ---- scatter, wide rows: one workgroup per row, the row assembled in LDS chunk by chunk -----------------
constexpr int kScatterChunk = 8192;  // columns per chunk (32 KiB of LDS)

template <typename IdxT, bool ALIGNED>
__global__ void __launch_bounds__(256)
    maxk_scatter_block_kernel(const float* __restrict__ grad_vals, const IdxT* __restrict__ idx, int64_t N, int M, int k,
                              float* __restrict__ grad_in) {
  __shared__ __attribute__((aligned(16))) float s_chunk[kScatterChunk];
  const int64_t r = blockIdx.x;
  if (r >= N) return;
  const float* gv = grad_vals + r * (int64_t)k;
  const IdxT* ix = idx + r * (int64_t)k;
  float* out = grad_in + r * (int64_t)M;
  int pad = ALIGNED ? 0 : floats_behind(out, 4);  // the first chunk is that much shorter, so that the others start on a boundary
  for (int c0 = 0; c0 < M;) {
    const int width = min(M - c0, kScatterChunk - pad);
    for (int q = threadIdx.x; q < pad + width; q += blockDim.x) s_chunk[q] = 0.0f;
    __syncthreads();
    for (int j = threadIdx.x; j < k; j += blockDim.x) {
      const int col = (int)ix[j] - c0;
      if ((unsigned)col < (unsigned)width) s_chunk[pad + col] = gv[j];
    }
    __syncthreads();
    store_image<ALIGNED>(out + c0, s_chunk, width, pad, (int)threadIdx.x, (int)blockDim.x);
    __syncthreads();  // the chunk buffer is zeroed again by the next round
    c0 += width;
    pad = 0;
  }
}

// ---- gather: the dense gradient row is read once, through LDS, with 128-bit loads ------------------------
//
// One wavefront per `rows` rows, at most kBackwardRowsM floats in all: 128-bit loads (from any 4-byte boundary, see load_group), four per lane at a
// time (eight: 2^20 x 256, k = 32 225 -> 219 us, 2^18 x 512 111.5 -> 109.2), then the saved columns' entries are read from LDS, and the results, again
// contiguous in the output, are stored coalesced.  FOURS: M is a multiple of four, so that nothing is left beside the 128-bit loads.
// twos: a full wavefront's rows, of 256, 512 or 1024 columns, are loaded two quads per lane at a time, without a look at the end.  With 65536 wavefronts and
// more and k from an eighth of the row on (four -> two, us: 2^20 x 256, k = 32 210.4 -> 206.6, inputs cold 223 -> 218, k = 128 358 -> 353, 2^18 x 1024 210.4 -> 206.5;
// but 528693 x 256, k = 11, byte columns 92.0 -> 95.6, 157978 x 256, k = 3 26.3 -> 28.5, 157897 x 512, k = 61 -1 %, 2^17 x 2048, k = 100, inputs cold, 190.3 -> 192.2,
// 2^20 x 64, k = 8 54.0 -> 55.9, and rows that share lines, 2^20 x 251 228 -> 230, 2^18 x 777 155 -> 163).
// FEW: a launch of few wavefronts, whose latencies stand alone: the columns are loaded before the rows.  Up to 32768 wavefronts of up to 400 pairs (last ->
// first, us: 3910 x 256, k = 15, byte columns 3.3 -> 2.9, 20000 x 64 3.2 -> 2.8, 1506 x 1028 4.0 -> 3.5, 48008 x 208 9.9 -> 9.1, 42280 x 256, k = 38 11.0 -> 10.0, of
// 16384 to 24575 wavefronts -2 % on average, to 32767 -0.5; but to 65535 +0.2, 2^20 x 256 210 -> 212 to 213, 2^20 x 251 226 -> 229, and more columns hold up the
// rows: 7632 x 832, k = 206 5.8 -> 6.2; as a flag to one kernel small launches take 0.03 to 0.05 us more).
template <typename IdxT, int BATCH, bool FOURS, bool FEW>
__device__ __forceinline__ void gather_rows(const float* __restrict__ grad_out, const IdxT* __restrict__ idx, int64_t N, int M, int k, int rows,
                                            int twos, uint32_t by, float* __restrict__ grad_vals) {
  extern __shared__ __attribute__((aligned(16))) float s_rows[];  // [rows * M], in whole quads
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
  const int lane = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  if (r0 >= N) return;
  const int nrows = rows_left(N - r0, rows), total = nrows * M, pairs = nrows * k, quads = total >> 2;
  const float* src = grad_out + r0 * (int64_t)M;
  const IdxT* ix = idx + r0 * (int64_t)k;
  float* to = grad_vals + r0 * (int64_t)k;
  constexpr int kQuads = kBackwardRowsM / 4 / kWave;
  int c[BATCH];
  auto load = [&](int p0) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) c[i] = (int)__builtin_nontemporal_load(ix + min(p0 + i * kWave + lane, pairs - 1));
  };
  if constexpr (FEW) load(0);
  float rest = 0.0f;
  if (!FOURS && lane < total - 4 * quads) rest = src[4 * quads + lane];
  auto copy = [&](auto at_once, auto full) {  // full: the rows fill the image
    constexpr int PART = decltype(at_once)::value;
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int part = 0; part < kQuads; part += PART) {
      if (FULL || part * kWave < quads) {  // uniform
        f4 v[PART];
#pragma unroll
        for (int i = 0; i < PART; ++i) {
          const int q = (part + i) * kWave + lane;
          v[i] = __builtin_nontemporal_load(reinterpret_cast<const f4_any*>(src) + (FULL ? q : min(q, quads - 1)));
        }
#pragma unroll
        for (int i = 0; i < PART; ++i) asm volatile("" : "+v"(v[i]));  // (or the loads move to their uses)
#pragma unroll
        for (int i = 0; i < PART; ++i) {
          const int q = (part + i) * kWave + lane;
          if (FULL || q < quads) reinterpret_cast<f4*>(s_rows)[q] = v[i];
        }
      }
    }
  };
  if (FOURS && !FEW && twos && quads == kQuads * kWave) {  // uniform
    copy(std::integral_constant<int, 2>(), std::true_type());
  } else {
    copy(std::integral_constant<int, 4>(), std::false_type());
  }
  if constexpr (!FEW) load(0);
  if (!FOURS && lane < total - 4 * quads) s_rows[4 * quads + lane] = rest;
  wavefront_lds_order();
  for (int p0 = 0;;) {
    float g[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const bool inside = (unsigned)c[i] < (unsigned)M;
      const float read = s_rows[inside ? quotient(min(p0 + i * kWave + lane, pairs - 1), by) * M + c[i] : 0];
      g[i] = inside ? read : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) asm volatile("" : "+v"(g[i]));
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int p = p0 + i * kWave + lane;
      if (p < pairs) to[p] = g[i];
    }
    p0 += BATCH * kWave;
    if (p0 >= pairs) break;
    load(p0);
  }
}

template <typename IdxT, int BATCH, bool FOURS>
__global__ void __launch_bounds__(kWave)
    maxk_gather_rows_kernel(const float* __restrict__ grad_out, const IdxT* __restrict__ idx, int64_t N, int M, int k, int rows,
                            int twos, uint32_t by, float* __restrict__ grad_vals) {
  gather_rows<IdxT, BATCH, FOURS, false>(grad_out, idx, N, M, k, rows, twos, by, grad_vals);
}
namespace few {
template <typename IdxT, int BATCH, bool FOURS>
__global__ void __launch_bounds__(kWave)
    maxk_gather_rows_kernel(const float* __restrict__ grad_out, const IdxT* __restrict__ idx, int64_t N, int M, int k, int rows,
                            int twos, uint32_t by, float* __restrict__ grad_vals) {
  gather_rows<IdxT, BATCH, FOURS, true>(grad_out, idx, N, M, k, rows, twos, by, grad_vals);
}
}  // namespace few

// ---- gather, wide rows: the saved columns are read straight from memory ---------------------------------
// (k scattered 4-byte reads per row; for k << M this touches far less than the whole row.)
template <typename IdxT>
__global__ void __launch_bounds__(256)
    maxk_gather_block_kernel(const float* __restrict__ grad_out, const IdxT* __restrict__ idx, int64_t N, int M, int k,
                             float* __restrict__ grad_vals) {
  const int64_t r = blockIdx.x;
  if (r >= N) return;
  const float* row = grad_out + r * (int64_t)M;
  for (int j = threadIdx.x; j < k; j += blockDim.x) {
    const int col = (int)idx[r * (int64_t)k + j];
    grad_vals[r * (int64_t)k + j] = (unsigned)col < (unsigned)M ? row[col] : 0.0f;
  }
}

// ---- host side --------------------------------------------------------------------------------------------


// Rows per wavefront of the gather: up to 8 KiB of LDS, fewer where that would leave compute units with less than four wavefronts (eight -> four, us:
// 3910 x 256, k = 15, byte columns 3.9 -> 3.3, 9824 x 64, k = 3 3.2 -> 3.0; eight where it has more than 400 pairs, 5098 x 384, k = 121 4.45 -> 4.2), but a
// 128-bit load for each lane.  A power of two of them where M is a multiple of four: wavefronts then seldom share a line of the rows, or of the results,
// which both would read, or write part of (as many as fit -> a power of two, us: 320696 x 88, k = 4 23 rows 24.2 -> 16 rows 20.7; 10^6 x 40, k = 2 51 34.2 -> 32 28.8; 500000 x 100, k = 12 20 43.4 -> 16 41.5;
// 300000 x 200 10 46.5 -> 8 44.2; 100000 x 400 5 29.5 -> 4 27.8; but odd widths, which share lines in any case: 100000 x 333 6 28.0 -> 4 29.0).  Of wider rows
// than 256 columns not where that takes more than a fifth of them (219907 x 644, k = 67 3 116.8 -> 2 123.8; 747932 x 288, k = 5 7 143 -> 4 150; 215027 x
// 516, k = 44 3 90.5 -> 2 94.9), unless it alone ends the results on a line (2^18 x 640, k = 80 3 141.9 -> 2 136.3).
constexpr int kFirstPairs = 400;  // (see gather_rows, too)
inline int backward_rows_per_wave(int64_t N, int M, int k) {
  const int most = kBackwardRowsM / M, least = 4 * kWave / M > 1 ? 4 * kWave / M : 1;
  auto spread = [&](int64_t wavefronts) { return N / wavefronts >= most ? most : (N / wavefronts > least ? (int)(N / wavefronts) : least); };
  int rows = spread(1024);
  if (rows * k > kFirstPairs) rows = spread(2048);
  const int power = 1 << (31 - __builtin_clz((unsigned)rows));
  return M % 4 == 0 && (M <= 256 || 5 * power >= 4 * rows || (power * k % 32 == 0 && rows * k % 32 != 0)) ? power : rows;
}

// f(integral_constant<int, BATCH>) for a wavefront of up to `pairs` pairs.  No more than it has: a load whose lanes are all past the end costs as
// much as another (1048576 x 256, k = 32, eight instructions of which four past the end 241 us, four 219).
template <typename F>
hipError_t by_pairs(int pairs, F f) {
  const int need = (pairs + kWave - 1) / kWave, times = (need + 15) / 16, each = (need + times - 1) / times;
#define X(n) if (each <= n) return f(std::integral_constant<int, n>());
  X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(13) X(16)
#undef X
  return hipErrorInvalidValue;  // not reached
}

template <typename IdxT>
hipError_t launch_scatter(const float* gv, const IdxT* idx, int64_t N, int M, int k, float* gin, hipStream_t stream) {
  if (M > kBackwardRowsM) {
    if (N > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const bool whole = M % 4 == 0 && floats_behind(gin, 4) == 0;  // (every row starts and ends on a boundary: 65536 x 3000 130 us, 137 without)
    return launch_kernel(whole ? maxk_scatter_block_kernel<IdxT, true> : maxk_scatter_block_kernel<IdxT, false>, dim3((unsigned)N), dim3(256), 0,
                         stream, gv, idx, N, M, k, gin);
  }
  const int64_t elements = N * M;
  int chunk = kBackwardRowsM;  // 8 KiB of LDS, less where that would leave compute units with less than eight wavefronts
  while (chunk > 512 && elements / chunk < 2048 - 2048 / 8) chunk >>= 1;
  const int skew = floats_behind(gin, 32);
  // Whole rows to a chunk where they end on lines, or where they have so many pairs that loading those of cut rows twice costs more than the lines that
  // two wavefronts write parts of.  The image is then smaller and the wavefronts are more, which very large outputs pay for (2048 floats -> whole rows,
  // us, inputs warm: 30774 x 1184, k = 304 35.5 -> 29.9, 25221 x 1600, k = 887 71 % of it, 13M elements 9596 x 1220, k = 631 80 %, 42M 21886 x 1928, k = 657
  // 79.5 %, k below 1 / 20 of the row 93 to 101 %; but 129M to 263M elements and small k 102 to 104 %, 151634 x 1456, k = 472 243 -> 268; with k from an eighth of
  // rows of more than 900 columns on 90 to 97 %, unless they leave a quarter of the 2048 floats, 197041 x 1088, k = 312 226.5 -> 242.5; ends beside lines, k =
  // M / 5 95 to 132 %, 38320 x 1004, k = 288, two rows to a chunk 37.7 -> 44.5).
  if (skew == 0 && M <= chunk &&
      (elements < 1 << 26 ? M % 32 == 0 || (M % 4 == 0 && M > 1024 && 4 * k >= M) : M % 32 == 0 && M > 900 && 8 * k >= M && chunk / M * M >= 1536))
    chunk = chunk / M * M;
  const int64_t blocks = (elements + skew + chunk - 1) / chunk;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const int whole = skew == 0 && chunk % M == 0 ? chunk / M : 0;
  const int rows = whole > 0 ? whole : (chunk + M - 2) / M + 1;  // that a chunk meets at most
  return by_pairs(rows * k, [&](auto batch) {
    constexpr int B = decltype(batch)::value;
    const bool stream_pairs = whole > 0 && whole * k * sizeof(IdxT) % 128 == 0;
    return launch_kernel(stream_pairs ? maxk_scatter_rows_kernel<IdxT, B, true> : maxk_scatter_rows_kernel<IdxT, B, false>,
                         dim3((unsigned)blocks), dim3(kWave), chunk * sizeof(float), stream, gv, idx, gin, elements, 1.0 / M, M, k, divisor(k), divisor(M),
                         (uint32_t)chunk | (uint32_t)skew << 12 | (uint32_t)whole << 17);
  });
}

template <typename IdxT>
hipError_t launch_gather(const float* gout, const IdxT* idx, int64_t N, int M, int k, float* gv, hipStream_t stream) {
  if (M > kBackwardRowsM) {
    if (N > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    return launch_kernel(maxk_gather_block_kernel<IdxT>, dim3((unsigned)N), dim3(256), 0, stream, gout, idx, N, M, k, gv);
  }
  const int rows = backward_rows_per_wave(N, M, k);
  const int64_t blocks = (N + rows - 1) / rows;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  return by_pairs(rows * k, [&](auto batch) {
    constexpr int B = decltype(batch)::value;
    const bool first = blocks < 32768 && rows * k <= kFirstPairs, twos = blocks >= 65536 && M % 256 == 0 && M <= 1024 && 8 * k >= M;  // (see gather_rows)
    const auto kernel = M % 4 == 0 ? (first ? few::maxk_gather_rows_kernel<IdxT, B, true> : maxk_gather_rows_kernel<IdxT, B, true>)
                                   : (first ? few::maxk_gather_rows_kernel<IdxT, B, false> : maxk_gather_rows_kernel<IdxT, B, false>);
    return launch_kernel(kernel, dim3((unsigned)blocks), dim3(kWave), ((size_t)rows * M + 3) / 4 * 16, stream, gout, idx, N, M, k, rows,
                         twos ? 1 : 0, divisor(k), gv);
  });
}

}  // namespace rtopk
