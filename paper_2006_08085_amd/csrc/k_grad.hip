// Local stochastic gradients of the synthetic objectives: the gradient query
// of Algorithm 2, every worker at its own model.
//
//   diagonal quadratic: G = h * (x - b_i) + sigma * z, z standard normal, either
//     read from an array or regenerated from the counter (seed, step, worker,
//     column) with Philox-4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and the
//     Box-Muller transform.  A thread owns the four columns of one Philox block.
//   least squares: G_i = A_i^T (A_i x_i - b_i), two small passes.
#include <algorithm>

#include "detag_internal.h"
#include "dev_common.hpp"
#include "fused_common.hpp"
#include "noise_dev.hpp"

namespace detag {
namespace {

constexpr int kThreads = 256;
// four columns are one access wherever the row starts (see k_stream.hip)
typedef float vf4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned short vu4_t __attribute__((ext_vector_type(4), aligned(2)));

template <bool NT>
__device__ __forceinline__ vf4_t load_wide(const vf4_t *p) { return NT ? __builtin_nontemporal_load(p) : *p; }
template <bool NT>
__device__ __forceinline__ vu4_t load_wide(const vu4_t *p) { return NT ? __builtin_nontemporal_load(p) : *p; }

// A block works on kGradRows consecutive worker rows of its 1024 columns, so that a shared curvature vector is
// read once per kGradRows rows instead of once per row (read per row it is a fourth stream: measured 1.33 x the
// bytes of X, b and G on 64 x 11.2 M).
constexpr int kGradRows = 4;

template <typename ST, bool NT>
__global__ __launch_bounds__(kThreads) void grad_quadratic_kernel(int n, int64_t d, int64_t ld, const ST *__restrict__ X,
                                                                  const float *__restrict__ h, int64_t h_row_stride,
                                                                  const float *__restrict__ b,
                                                                  const float *__restrict__ noise, float sigma,
                                                                  uint32_t seed_lo, uint32_t seed_hi, uint32_t step,
                                                                  float *__restrict__ G) {
  const int64_t q = int64_t(blockIdx.x) * kThreads + threadIdx.x;  // Philox block = 4 columns
  const int64_t c0 = q * 4;
  if (c0 >= d) return;
  const int i0 = blockIdx.y * kGradRows;
  const int valid = int(d - c0 < 4 ? d - c0 : 4);
  const bool wide = valid == 4;
  float hs[4] = {0.f, 0.f, 0.f, 0.f};
  if (h_row_stride == 0) {  // shared by the workers: read once, cached (other blocks read it too)
    if (wide) {
      const vf4_t th = *reinterpret_cast<const vf4_t *>(h + c0);
      hs[0] = th.x, hs[1] = th.y, hs[2] = th.z, hs[3] = th.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) hs[e] = e < valid ? h[c0 + e] : 0.f;
    }
  }
#pragma unroll
  for (int r = 0; r < kGradRows; ++r) {
    const int i = i0 + r;
    if (i >= n) break;
    const int64_t off = int64_t(i) * ld + c0;
    float x[4], hv[4], bv[4], z[4] = {0.f, 0.f, 0.f, 0.f};
    if (wide) {
      // b, the noise array, per-worker curvature and G are touched once: large calls stream them.  X never: the step that
      // follows reads it again, and finds what the memory-side cache kept of it (this call and a step with K = 4, 64
      // workers, 4-regular, fp32, three states in turn: d = 300,000 140 -> 132 us, 1,000,000 428 -> 389, 2,000,000 852 ->
      // 812; D-PSGD 87 -> 82, 272 -> 241, 550 -> 509).  The round of Algorithm 1 does not read X again: streamed and not, 139.5
      // and 140.6, 442.6 and 444.7, 885.3 and 884.2; 300 workers, d = 200,000, factor by factor, 1395 and 1399.
      if constexpr (sizeof(ST) == 4) {
        const vf4_t t = load_wide<false>(reinterpret_cast<const vf4_t *>(X + off));
        x[0] = t.x, x[1] = t.y, x[2] = t.z, x[3] = t.w;
      } else {
        const vu4_t t = load_wide<false>(reinterpret_cast<const vu4_t *>(X + off));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(uint32_t(t[e]) << 16);
      }
      const vf4_t tb = load_wide<NT>(reinterpret_cast<const vf4_t *>(b + off));
      bv[0] = tb.x, bv[1] = tb.y, bv[2] = tb.z, bv[3] = tb.w;
      if (h_row_stride) {
        const vf4_t th = load_wide<NT>(reinterpret_cast<const vf4_t *>(h + int64_t(i) * h_row_stride + c0));
        hv[0] = th.x, hv[1] = th.y, hv[2] = th.z, hv[3] = th.w;
      }
      if (noise) {
        const vf4_t tz = load_wide<NT>(reinterpret_cast<const vf4_t *>(noise + off));
        z[0] = tz.x, z[1] = tz.y, z[2] = tz.z, z[3] = tz.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = e < valid;
        x[e] = ok ? to_f32(X[off + e]) : 0.f;
        if (h_row_stride) hv[e] = ok ? h[int64_t(i) * h_row_stride + c0 + e] : 0.f;
        bv[e] = ok ? b[off + e] : 0.f;
        if (noise) z[e] = ok ? noise[off + e] : 0.f;
      }
    }
    if (!h_row_stride) {
#pragma unroll
      for (int e = 0; e < 4; ++e) hv[e] = hs[e];
    }
    if (!noise && sigma != 0.f) normal4(uint64_t(q), uint32_t(i), step, seed_lo, seed_hi, z);
    float g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = fmaf(sigma, z[e], hv[e] * (x[e] - bv[e]));
    if (wide) {
      const vf4_t tg = {g[0], g[1], g[2], g[3]};
      __builtin_nontemporal_store(tg, reinterpret_cast<vf4_t *>(G + off));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < valid) G[off + e] = g[e];
    }
  }
}

__device__ __forceinline__ vf4_t load4(const float *p) { return *reinterpret_cast<const vf4_t *>(p); }
__device__ __forceinline__ vf4_t load4(const bf16_t *p) {
  const vu4_t t = *reinterpret_cast<const vu4_t *>(p);
  vf4_t v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(uint32_t(t[e]) << 16);
  return v;
}

// acc[q][k] += the products of row q and x, pieces k, k + 4, ... of 256 columns, for ROWS rows side by side: a lane takes four
// columns of a piece, and the loads of four pieces are in flight.  In the last d % 1024 columns a lane whose four do not all
// exist takes the row's last four and leaves those out that are not its own (column by column, 64 at a time, their loads
// waited for one another: 8 workers, 64 x 1000 10.4 us in one launch, so 7.1; 32, 33 x 777 6.0 us for the first of two, so
// 3.6; 16, 100 x 4999 11.0, so 8.0).
constexpr int kPieces = 4;
template <int ROWS, typename ST>
__device__ __forceinline__ void lstsq_dot(const float *const (&row)[ROWS], const ST *x, int64_t d, int lane,
                                          float (&acc)[ROWS][kPieces]) {
  int64_t c = lane * 4;
  vf4_t av[ROWS][kPieces], xv[kPieces];
  auto add = [&](int k) {
#pragma unroll
    for (int q = 0; q < ROWS; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[q][k] = fmaf(av[q][k][e], xv[k][e], acc[q][k]);
  };
  for (; c - lane * 4 + kPieces * 256 <= d; c += kPieces * 256) {
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      xv[k] = load4(x + c + 256 * k);
#pragma unroll
      for (int q = 0; q < ROWS; ++q) av[q][k] = load4(row[q] + c + 256 * k);
    }
#pragma unroll
    for (int k = 0; k < kPieces; ++k) add(k);
  }
  const int left = int(d - (c - lane * 4));  // uniform, < 1024
  if (d < 4) {
    if (lane < left) {
#pragma unroll
      for (int q = 0; q < ROWS; ++q) acc[q][0] = fmaf(row[q][lane], to_f32(x[lane]), acc[q][0]);
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kPieces; ++k)
    if (256 * k < left) {
      const int64_t own = c + 256 * k, at = own < d - 4 ? own : d - 4;
      const int skip = int(own - at);
      xv[k] = load4(x + at);
#pragma unroll
      for (int q = 0; q < ROWS; ++q) av[q][k] = load4(row[q] + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) xv[k][e] = e < skip ? 0.f : xv[k][e];
#pragma unroll
      for (int q = 0; q < ROWS; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) av[q][k][e] = e < skip ? 0.f : av[q][k][e];
    }
#pragma unroll
  for (int k = 0; k < kPieces; ++k)
    if (256 * k < left) add(k);
}

// resid[i*m + r] = A_i[r,:] . x_i - b_i[r]; one block of one wavefront per (i, r), which spreads a few hundred rows over
// all compute units.  Four 16-byte pieces of the row and of x are in flight per lane, each with a sum of its own.
template <typename ST>
__global__ __launch_bounds__(64) void lstsq_resid_kernel(int64_t first_row, int m, int64_t d, int64_t ld, const ST *__restrict__ X,
                                                         const float *__restrict__ A, const float *__restrict__ b,
                                                         float *__restrict__ resid) {
  const int64_t row = first_row + blockIdx.x;  // = i*m + r
  const int lane = threadIdx.x;
  const float *a = A + row * d;
  const ST *x = X + (row >> 32 ? row / m : int64_t(uint32_t(row) / uint32_t(m))) * ld;
  const float target = b[row];  // not behind the sum
  float acc[1][kPieces] = {};
  const float *const only[1] = {a};
  lstsq_dot(only, x, d, lane, acc);
  float sum = (acc[0][0] + acc[0][1]) + (acc[0][2] + acc[0][3]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o, 64);
  if (lane == 0) resid[row] = sum - target;
}

// G[i,c] = sum_r A_i[r,c] * resid[i,r].  A block owns 4 * LANES columns of one worker; LANES lanes side by side take a
// row, so its 16 wavefronts walk 1024 / LANES rows at a time and add their parts up at the end.  With 16 lanes (64
// columns) a small problem makes enough blocks and a row of 64 samples is one step; with 64 lanes a wavefront reads 1 KiB
// of a row.
constexpr int kSumThreads = 1024;
template <int LANES>
__device__ __forceinline__ void lstsq_columns(const float *a, const float *res, int m, int64_t d, int64_t c, int r0, int lane,
                                              float (*part)[4 * LANES]) {
  constexpr int kRows = kSumThreads / LANES;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (c + 4 <= d) {
#pragma unroll 4
    for (int r = r0; r < m; r += kRows) {
      const vf4_t v = load4(a + int64_t(r) * d + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(v[e], res[r], acc[e]);
    }
  } else {
    for (int r = r0; r < m; r += kRows)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < d) acc[e] = fmaf(a[int64_t(r) * d + c + e], res[r], acc[e]);
  }
#pragma unroll
  for (int o = LANES; o < 64; o <<= 1)  // rows of one wavefront
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  if ((threadIdx.x & 63) < LANES) {
#pragma unroll
    for (int e = 0; e < 4; ++e) part[threadIdx.x >> 6][4 * lane + e] = acc[e];
  }
  __syncthreads();
}
template <int COLS>
__device__ __forceinline__ float lstsq_total(const float (*part)[COLS], int col) {
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < kSumThreads / 64; ++w) sum += part[w][col];
  return sum;
}

template <int LANES>
__global__ __launch_bounds__(kSumThreads) void lstsq_grad_kernel(int64_t first_col, int m, int64_t d, int64_t ld,
                                                                 const float *__restrict__ A, const float *__restrict__ resid,
                                                                 float *__restrict__ G) {
  constexpr int kCols = 4 * LANES, kWaves = kSumThreads / 64;
  __shared__ float part[kWaves][kCols];
  const int i = blockIdx.y, lane = threadIdx.x % LANES, r0 = threadIdx.x / LANES;
  const int64_t c0 = first_col + int64_t(blockIdx.x) * kCols;
  lstsq_columns<LANES>(A + int64_t(i) * m * d, resid + int64_t(i) * m, m, d, c0 + 4 * lane, r0, lane, part);
  if (threadIdx.x < kCols && c0 + threadIdx.x < d) G[int64_t(i) * ld + c0 + threadIdx.x] = lstsq_total(part, threadIdx.x);
}

// Both products in one launch, for problems so small that a block of 64 columns computes all residuals of its worker itself,
// in one go: a wavefront per row as in lstsq_resid_kernel, whose sums they are bit for bit, kSumRows rows side by side.  What
// such a call costs is the host behind its launches, not the GPU.  With a step after it, called back to back, two launches and
// one: 8 workers, 64 x 512 9.6 and 7.6 us, 64 x 1024 9.4 and 9.0, 16 x 1024 9.7 and 8.6, 16 workers, 64 x 768 9.4 and 9.2, 32,
// 64 x 384 9.7 and 9.5; on the GPU (replayed, the gradient alone) they take 5.2 and 5.2, 5.3 and 6.3, 4.9 and 5.9, 5.7 and 6.0,
// 5.7 and 5.4.  Blocks of a worker go to one XCD where n is a multiple of eight, so that its L2 serves all of them but the
// first.  Blocks of 128 and 256 columns repeat less of the first product and are slower both ways (8 workers, 64 x 1024 6.8
// and 8.7 us a call then).
constexpr int kSumRows = 4;
constexpr int kSmallRows = kSumRows * (kSumThreads / 64), kSmallCols = 1024;
template <typename ST>
__global__ __launch_bounds__(kSumThreads) void lstsq_small_kernel(int m, int64_t d, int64_t ld, const ST *__restrict__ X,
                                                                  const float *__restrict__ A, const float *__restrict__ b,
                                                                  float *__restrict__ G) {
  constexpr int kLanes = 16, kCols = 4 * kLanes, kWaves = kSumThreads / 64;
  __shared__ float res[kSmallRows];
  __shared__ float part[kWaves][kCols];
  const int i = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const float *a = A + int64_t(i) * m * d;
  const ST *x = X + int64_t(i) * ld;
  {
    const int r0 = wave < m ? wave : 0;  // rows past the last repeat another one
    float acc[kSumRows][kPieces] = {};
    const float *row[kSumRows];
#pragma unroll
    for (int q = 0; q < kSumRows; ++q) row[q] = a + int64_t(wave + q * kWaves < m ? wave + q * kWaves : r0) * d;
    lstsq_dot(row, x, d, lane, acc);
#pragma unroll
    for (int q = 0; q < kSumRows; ++q) {
      float sum = (acc[q][0] + acc[q][1]) + (acc[q][2] + acc[q][3]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o, 64);
      const int r = wave + q * kWaves;
      if (lane == 0 && r < m) res[r] = sum - b[int64_t(i) * m + r];
    }
  }
  __syncthreads();
  const int l = threadIdx.x % kLanes, r0 = threadIdx.x / kLanes;
  const int64_t c0 = int64_t(blockIdx.y) * kCols;
  lstsq_columns<kLanes>(a, res, m, d, c0 + 4 * l, r0, l, part);
  if (threadIdx.x < kCols && c0 + threadIdx.x < d) G[int64_t(i) * ld + c0 + threadIdx.x] = lstsq_total(part, threadIdx.x);
}

// One launch while a block takes its rows in one go, the blocks take a compute unit each and what they repeat of the first
// product stays small (with a step after it, called back to back, two launches and one: 16 workers, 64 x 900 9.6 and 10.4 us,
// 64 x 1024 9.2 and 9.7, which repeat 14 and 17 million products; 16, 64 x 768 and 32, 64 x 512, 9.4 and 8.4 million, are within
// 3 %).  With twice the rows or columns it is slower on the GPU by more than the launch it saves (16 workers, 64 x 2048 6.8 and
// 15.7 us a call, 8, 64 x 2000 6.2 and 9.1).
// A recorded call costs the host nothing at its replay and takes what is faster on the GPU: one launch up to 256 columns (two and
// one: 8 workers, 32 x 200 4.8 and 4.5 us, 64 workers, 64 x 256 6.1 and 4.9, 85, 40 x 129 5.8 and 4.8), from there to 512 either
// (8, 64 x 300 with the step 8.0 and 8.0, 512 7.6 and 7.8, 32, 64 x 384 9.9 and 9.5), then two (8, 64 x 640 8.2 and 8.5, 1024
// 7.7 and 8.8).
constexpr int kRecordedCols = 256;
constexpr int64_t kRepeated = int64_t(10) << 20;
bool lstsq_is_small(const Shape &s, int m, void *stream) {
  const int64_t blocks = (s.d + 63) / 64 * s.n;
  return m <= kSmallRows && s.d <= kSmallCols && blocks <= 256 && blocks * m * s.d <= kRepeated &&
         (s.d <= kRecordedCols || !is_capturing(stream));
}

bool overlap(const void *p, size_t p_bytes, const void *q, size_t q_bytes) {
  const auto a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
  return a < b + q_bytes && b < a + p_bytes;
}
// Whether G lies over X or b.  Two launches have read both before the second writes G; in the one launch a block writes its
// columns while others still read.
bool lstsq_in_place(const Shape &s, const void *X, const float *b, int m, const float *G) {
  const size_t elements = size_t(s.n - 1) * s.ld + s.d;
  return overlap(G, elements * 4, X, elements * (s.bf16 ? 2 : 4)) || overlap(G, elements * 4, b, size_t(s.n) * m * 4);
}

}  // namespace

int launch_grad_quadratic(const Shape &s, const void *X, const float *h, int h_per_worker, const float *b,
                          const float *noise, float sigma, uint64_t seed, uint32_t step, float *G, void *stream) {
  const int64_t blocks4 = (s.d + 3) / 4;
  const dim3 grid(ceil_div_i64(blocks4, kThreads), (s.n + kGradRows - 1) / kGradRows);
  auto st = static_cast<hipStream_t>(stream);
  const int64_t hstride = h_per_worker ? s.ld : 0;
  const uint32_t slo = uint32_t(seed & 0xffffffffu), shi = uint32_t(seed >> 32);
  auto go = [&](auto *kernel, auto *x) {
    kernel<<<grid, kThreads, 0, st>>>(s.n, s.d, s.ld, x, h, hstride, b, noise, sigma, slo, shi, step, G);
  };
  const bool nt = fused::loads_stream(s, (s.bf16 ? 2 : 4) + 8 + (h_per_worker ? 4 : 0) + (noise ? 4 : 0));
  auto with = [&](auto *x) {
    using ST = std::remove_const_t<std::remove_pointer_t<decltype(x)>>;
    go(nt ? &grad_quadratic_kernel<ST, true> : &grad_quadratic_kernel<ST, false>, x);
  };
  if (s.bf16) with(static_cast<const bf16_t *>(X));
  else with(static_cast<const float *>(X));
  return hip_rc(hipGetLastError());
}

int launch_grad_lstsq(const Shape &s, const void *X, const float *A, const float *b, int m, float *resid, float *G,
                      void *stream) {
  auto st = static_cast<hipStream_t>(stream);
  const int64_t rows = int64_t(s.n) * m;
  if (lstsq_is_small(s, m, stream) && !lstsq_in_place(s, X, b, m, G)) {
    const dim3 grid(s.n, ceil_div_i64(s.d, 64));
    if (s.bf16) lstsq_small_kernel<bf16_t><<<grid, kSumThreads, 0, st>>>(m, s.d, s.ld, static_cast<const bf16_t *>(X), A, b, G);
    else lstsq_small_kernel<float><<<grid, kSumThreads, 0, st>>>(m, s.d, s.ld, static_cast<const float *>(X), A, b, G);
    return hip_rc(hipGetLastError());
  }
  for (int64_t first = 0; first < rows; first += kThreadsPerLaunch / 64) {
    const dim3 grid(uint32_t(std::min(rows - first, kThreadsPerLaunch / 64)));
    if (s.bf16)
      lstsq_resid_kernel<bf16_t><<<grid, 64, 0, st>>>(first, m, s.d, s.ld, static_cast<const bf16_t *>(X), A, b, resid);
    else
      lstsq_resid_kernel<float><<<grid, 64, 0, st>>>(first, m, s.d, s.ld, static_cast<const float *>(X), A, b, resid);
    if (int rc = hip_rc(hipGetLastError())) return rc;
  }
  // 64 columns per block until blocks of 256 columns alone make two per compute unit
  if (int64_t(ceil_div_i64(s.d, 256)) * s.n < 512) {
    lstsq_grad_kernel<16><<<dim3(ceil_div_i64(s.d, 64), s.n), kSumThreads, 0, st>>>(0, m, s.d, s.ld, A, resid, G);
    return hip_rc(hipGetLastError());
  }
  constexpr int64_t kPiece = kThreadsPerLaunch / kSumThreads * 256;  // columns
  for (int64_t first = 0; first < s.d; first += kPiece) {
    const dim3 grid(ceil_div_i64(std::min(s.d - first, kPiece), 256), s.n);
    lstsq_grad_kernel<64><<<grid, kSumThreads, 0, st>>>(first, m, s.d, s.ld, A, resid, G);
    if (int rc = hip_rc(hipGetLastError())) return rc;
  }
  return 0;
}

}  // namespace detag
