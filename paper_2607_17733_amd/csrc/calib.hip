// calib.hip -- on-GPU calibration: the offline step that produces the
// path's inputs, the column permutation and the per-block width map.
//
// MXSens (arXiv 2607.17733), Section 3, Algorithm 1: a column's sensitivity
// is the diagonal of the Hessian approximation H = sum over calibration
// samples of X^T X, i.e. the sum of its squared activations.  Section 4.2,
// Algorithm 2: sort a layer's columns by descending sensitivity; the top 32
// get 8-bit mantissas, the next N6 6-bit, the rest 4-bit.
//
// Sensitivities are float64 and computed in a fixed order, one lane per
// column: a sample's rows are summed in row order from zero (every square of
// a bf16 value is exact in float64), and the sample's sum is then added to
// the running total.  The row order makes each column one serial chain of
// float64 additions, so the parallelism is columns x samples: one lane per
// column and sample, all samples of a call in one launch.  The sort is by
// counting: a column's rank is the number of columns that sort before it
// (larger sensitivity, or equal with a lower index; a NaN counts as +inf),
// which fixes a unique order without a parallel sort.  The rank then places
// the column in the permutation: the 4-bit columns first, then the 6-bit and
// the 8-bit ones, each in sorted order.
#include "mxq_internal.h"
#include <algorithm>
#include <type_traits>

namespace mxq {

namespace {

constexpr int kCalThreads = 256;

__device__ inline double bf16_to_f64(uint16_t v) {
  return (double)__uint_as_float((uint32_t)v << 16);
}

// The samples of one launch: sample i's rows start at x[i], or, for a batch
// in one tensor, at base + i * stride.
struct SampleList {
  const uint16_t *x[MXQ_CALIB_LIST_MAX];
  int64_t rows[MXQ_CALIB_LIST_MAX], ld[MXQ_CALIB_LIST_MAX];
};
struct SampleBatch {
  const uint16_t *base;
  int64_t stride, nrows, lead;
};
__device__ inline const uint16_t *sample_ptr(const SampleList &l, int i) { return l.x[i]; }
__device__ inline int64_t sample_rows(const SampleList &l, int i) { return l.rows[i]; }
__device__ inline int64_t sample_ld(const SampleList &l, int i) { return l.ld[i]; }
__device__ inline const uint16_t *sample_ptr(const SampleBatch &b, int i) {
  return b.base + (int64_t)i * b.stride;
}
__device__ inline int64_t sample_rows(const SampleBatch &b, int) { return b.nrows; }
__device__ inline int64_t sample_ld(const SampleBatch &b, int) { return b.lead; }

// A lane per column, COLS columns per workgroup (blockIdx.x) and sample
// (blockIdx.y): the column sums of the sample in row order, to its row of
// `out` (or added to it).  A wave keeps the next BATCH rows in flight while it
// sums the current ones; the rows left over are one more such set (2047 x 4096:
// 41.9 us, read one after the other 51.3).  The kernel is bound by the HBM read
// once enough rows are in flight: few waves need 32 each (64 loads, the most a wave can count),
// and one wave per workgroup to spread over the CUs; more than 8 per CU do with
// 4 each, and workgroups of 256 adjacent columns read longer runs.  Sixteen
// samples of 2048 x 4096 (268 MB): 43.5 us (6.2 TB/s; a launch per sample, whose
// 64 waves are a sixteenth of the GPU's SIMDs, took 98 us each, a batch with 8
// rows in flight 107); 128 samples 388 us with 4 rows, 401 with 32, 449 with 32
// and 64 columns per workgroup.
template <class Samples, int COLS, int BATCH>
__global__ __launch_bounds__(COLS) void colsq_kernel(Samples sm, int64_t K, double *out,
                                                     int accumulate) {
  const int y = blockIdx.y;
  const int64_t k = (int64_t)blockIdx.x * COLS + threadIdx.x;
  const int64_t rows = sample_rows(sm, y), ld = sample_ld(sm, y);
  if (k >= K) return;
  const uint16_t *p = sample_ptr(sm, y) + k;
  double sum = 0.0;
  auto fetch = [&](uint16_t (&v)[BATCH], int64_t r) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = p[(r + u) * ld];
  };
  auto add = [&](const uint16_t (&v)[BATCH]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const double d = bf16_to_f64(v[u]);
      sum += d * d;
    }
  };
  const int64_t nb = rows / BATCH;
  if (nb > 0) {
    uint16_t a[BATCH], b[BATCH];
    fetch(a, 0);
    int64_t i = 1;
    for (; i + 1 < nb; i += 2) {
      fetch(b, i * BATCH);
      add(a);
      fetch(a, (i + 1) * BATCH);
      add(b);
    }
    if (i < nb) {
      fetch(b, i * BATCH);
      add(a);
      add(b);
    } else {
      add(a);
    }
  }
  // the rows left over, their loads in flight together too: those of the 1, 8 or
  // BATCH loads that lie past the end repeat the last row and add 0 (exact: the
  // sum is never -0)
  const int rem = (int)(rows - nb * BATCH);
  auto left = [&](auto n) __attribute__((always_inline)) {
    constexpr int N = decltype(n)::value;
    uint16_t v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = p[(nb * BATCH + min(u, rem - 1)) * ld];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const double d = u < rem ? bf16_to_f64(v[u]) : 0.0;
      sum += d * d;
    }
  };
  if (rem > 8)
    left(std::integral_constant<int, BATCH>{});
  else if (rem > 1)
    left(std::integral_constant<int, (BATCH < 8 ? BATCH : 8)>{});
  else if (rem == 1)
    left(std::integral_constant<int, 1>{});
  double *o = out + (int64_t)y * K + k;
  *o = accumulate ? *o + sum : sum;
}

__global__ __launch_bounds__(kCalThreads) void add_samples_kernel(const double *__restrict__ part,
                                                                  int64_t n, int64_t K, double *s,
                                                                  int accumulate) {
  const int64_t k = (int64_t)blockIdx.x * kCalThreads + threadIdx.x;
  if (k >= K) return;
  double acc = accumulate ? s[k] + part[k] : part[k];
  for (int64_t i = 1; i < n; ++i) acc = acc + part[i * K + k];
  s[k] = acc;
}

__device__ inline double sort_key(double v) { return v != v ? __builtin_inf() : v; }

// A workgroup ranks kRankCols columns; each wave compares 64 columns j at a
// time with all of them.  The compare leaves a lane mask, whose population
// count is scalar work, so a (column, 64 j) pair costs one vector
// instruction: the rank of K columns is K^2 / 64 compares spread over
// K / kRankCols workgroups (K = 4096: 8.9 us; one thread per column, sixteen
// workgroups walking all K keys, took 310 us).
// PRE sets of 64 columns a wave has in flight: 8 for long rows, no more than
// there are for short ones (K = 32: 8 sets 5.9 us, 1 set 4.0).
constexpr int kRankCols = 16;

template <int PRE>
__global__ __launch_bounds__(kCalThreads) void rank_perm_kernel(const double *__restrict__ s,
                                                                int64_t K, int64_t n4,
                                                                int64_t n6, int64_t n8,
                                                                int32_t *perm) {
  constexpr int kW = kCalThreads / 64;
  __shared__ int cnt[kW][kRankCols];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * kRankCols;
  double key[kRankCols];
  int before[kRankCols];
#pragma unroll
  for (int c = 0; c < kRankCols; ++c) {
    key[c] = i0 + c < K ? sort_key(s[i0 + c]) : 0.0;
    before[c] = 0;
  }
  // 64 columns from j0: all of them before the workgroup's columns (equal
  // sensitivities sort first), all after, or mixed.  The loads of PRE such
  // sets are issued together: one after the other they were most of the time.
  for (int64_t jb = 64 * wave; jb < K; jb += PRE * kCalThreads) {
    double raw[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int64_t j = jb + u * kCalThreads + lane;
      raw[u] = s[j < K ? j : K - 1];
    }
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int64_t j0 = jb + u * kCalThreads, j = j0 + lane;
      const bool in = j < K;
      const double sj = in ? sort_key(raw[u]) : -__builtin_inf();   // not before any column
      if (j0 + 64 <= i0) {
#pragma unroll
        for (int c = 0; c < kRankCols; ++c) before[c] += __popcll(__ballot(sj >= key[c]));
      } else if (j0 >= i0 + kRankCols) {
#pragma unroll
        for (int c = 0; c < kRankCols; ++c) before[c] += __popcll(__ballot(sj > key[c]));
      } else {
#pragma unroll
        for (int c = 0; c < kRankCols; ++c)
          before[c] += __popcll(__ballot(in && (sj > key[c] || (sj == key[c] && j < i0 + c))));
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kRankCols; ++c)
    if (lane == 0) cnt[wave][c] = before[c];
  __syncthreads();
  const int64_t i = i0 + threadIdx.x;
  if (threadIdx.x >= kRankCols || i >= K) return;
  int64_t rank = 0;
#pragma unroll
  for (int w = 0; w < kW; ++w) rank += cnt[w][threadIdx.x];
  const int64_t c8 = 32 * n8, c6 = 32 * n6, c4 = 32 * n4;
  int64_t pos;
  if (rank < c8) pos = c4 + c6 + rank;                       // 8-bit: the last blocks
  else if (rank < c8 + c6) pos = c4 + (rank - c8);           // 6-bit
  else pos = rank - c8 - c6;                                 // 4-bit: the first blocks
  perm[pos] = (int32_t)i;
}

// max_rows: the rows of the longest sample.  Below 64 rows a wave has no whole
// pair of batches to overlap, and 64 columns per workgroup only make more
// workgroups (sixteen samples of 31 x 4096: 9.3 us, wide ones 6.7; of 100 x 4096
// 12.6 and 12.6, of 300 18.4 and 29.7).
template <class Samples>
hipError_t go_colsq(const Samples &sm, int64_t n, int64_t max_rows, int64_t K, double *out,
                    bool accumulate, hipStream_t stream) {
  auto launch = [&](auto fn, int cols) {
    hipLaunchKernelGGL(fn, dim3((unsigned)((K + cols - 1) / cols), (unsigned)n), dim3(cols), 0,
                       stream, sm, K, out, accumulate ? 1 : 0);
  };
  if (max_rows >= 64 && (K + 63) / 64 * n <= 8 * (int64_t)device_cu_count())
    launch(colsq_kernel<Samples, 64, 32>, 64);
  else
    launch(colsq_kernel<Samples, 256, 4>, 256);
  return hipGetLastError();
}

hipError_t go_add(const double *part, int64_t n, int64_t K, double *s, bool accumulate,
                  hipStream_t stream) {
  const int64_t blocks = (K + kCalThreads - 1) / kCalThreads;
  hipLaunchKernelGGL(add_samples_kernel, dim3((unsigned)blocks), dim3(kCalThreads), 0, stream,
                     part, n, K, s, accumulate ? 1 : 0);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_calib_colsq(const uint16_t *x, int64_t rows, int64_t ld, int64_t K, double *s,
                              bool accumulate, hipStream_t stream) {
  return go_colsq(SampleBatch{x, 0, rows, ld}, 1, rows, K, s, accumulate, stream);
}

hipError_t launch_calib_colsq_samples(const uint16_t *x, int64_t n, int64_t rows, int64_t ld,
                                      int64_t sample_stride, int64_t K, double *part, double *s,
                                      bool accumulate, hipStream_t stream) {
  const hipError_t e = go_colsq(SampleBatch{x, sample_stride, rows, ld}, n, rows, K, part,
                                false, stream);
  return e != hipSuccess ? e : go_add(part, n, K, s, accumulate, stream);
}

hipError_t launch_calib_colsq_list(const uint16_t *const *x, const int64_t *rows,
                                   const int64_t *ld, int64_t n, int64_t K, double *part,
                                   double *s, bool accumulate, hipStream_t stream) {
  SampleList l{};
  int64_t max_rows = 0;
  for (int64_t i = 0; i < n; ++i) {
    l.x[i] = x[i];
    l.rows[i] = rows[i];
    max_rows = std::max(max_rows, rows[i]);
    l.ld[i] = ld[i];
  }
  const hipError_t e = go_colsq(l, n, max_rows, K, part, false, stream);
  return e != hipSuccess ? e : go_add(part, n, K, s, accumulate, stream);
}

hipError_t launch_calib_perm(const double *s, int64_t K, int64_t n6, int64_t n8, int32_t *perm,
                             hipStream_t stream) {
  const int64_t blocks = (K + kRankCols - 1) / kRankCols;
  const auto fn = K <= kCalThreads       ? rank_perm_kernel<1>
                  : K <= 4 * kCalThreads ? rank_perm_kernel<4>
                                         : rank_perm_kernel<8>;
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kCalThreads), 0, stream, s,
                     K, K / 32 - n6 - n8, n6, n8, perm);
  return hipGetLastError();
}

}  // namespace mxq
