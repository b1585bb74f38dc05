// Diagnostics: the worker mean (the output line of Algorithm 2) and the
// consensus distance ||X - 1 xbar^T||_F^2 bounded in the proof of Theorem 3.
// One lane owns one column and walks the n rows once; sums are kept in fp64 and
// taken relative to the first worker's value, so the distance stays meaningful
// when the workers almost agree.  Reductions use a
// fixed order (wavefront shuffle tree, then one block over the per-block
// partials): results are bit-reproducible.
#include "dev_common.hpp"
#include "detag_internal.h"
#include "fused_common.hpp"

namespace detag {
namespace {

constexpr int kThreads = 256;

// X is read once per kernel: non-temporal where the call streams (fused::tile_access; worker mean and consensus distance of
// 64 x 1,000,003, pitch d, fp32 50 and 57 us streamed, 47 and 54 not, bf16 29 and 41, 25 and 35; on lines 43 and 51, 46 and
// 53; 16 x 272,474, which the caches keep, distance 13 and 10).
template <bool NT>
__device__ __forceinline__ float load_f32(const float *p) { return NT ? __builtin_nontemporal_load(p) : *p; }
template <bool NT>
__device__ __forceinline__ float load_f32(const bf16_t *p) {
  return __uint_as_float(uint32_t(NT ? __builtin_nontemporal_load(&p->bits) : p->bits) << 16);
}

template <typename ST, bool NT>
__global__ __launch_bounds__(kThreads) void mean_kernel(int n, int64_t d, int64_t ld, const ST *__restrict__ X,
                                                        float *__restrict__ xbar) {
  const int64_t c = int64_t(blockIdx.x) * kThreads + threadIdx.x;
  if (c >= d) return;
  double s = 0.0;
#pragma unroll 16
  for (int i = 0; i < n; ++i) s += double(load_f32<NT>(X + int64_t(i) * ld + c));  // 16 rows' loads in flight
  __builtin_nontemporal_store(float(s / n), xbar + c);  // 64 x 11.2 M: 465 us with a plain store, 453 so; up to 64 x 1,000,000 the same
}

template <int THREADS = kThreads>
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double part[THREADS / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < THREADS / 64; ++w) t += part[w];
  return t;  // valid in thread 0
}

template <typename ST, bool NT>
__global__ __launch_bounds__(kThreads) void consensus_partial_kernel(int n, int64_t d, int64_t ld,
                                                                     const ST *__restrict__ X,
                                                                     double *__restrict__ partials) {
  const int64_t c = int64_t(blockIdx.x) * kThreads + threadIdx.x;
  double acc = 0.0;
  if (c < d) {
    // One pass: with e_i = x_i - x_0 (exact in fp64 for fp32 or bf16 inputs),
    //   sum_i (x_i - mean)^2 = sum_i e_i^2 - (sum_i e_i)^2 / n.
    // Both terms are of the size of the result (the shift by x_0 removes the common part of the column), so the
    // subtraction does not cancel, however close the workers are to agreement.
    const double x0 = double(load_f32<NT>(X + c));
    double s1 = 0.0, s2 = 0.0;
#pragma unroll 16
    for (int i = 1; i < n; ++i) {
      const double e = double(load_f32<NT>(X + int64_t(i) * ld + c)) - x0;
      s1 += e;
      s2 = fma(e, e, s2);
    }
    acc = s2 - s1 * s1 / n;
    acc = acc < 0.0 ? 0.0 : acc;
  }
  const double t = block_sum(acc);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

constexpr int kSumThreads = 1024;
__global__ __launch_bounds__(kSumThreads) void sum_partials_kernel(int64_t count, const double *__restrict__ partials,
                                                                   double *__restrict__ out) {
  // eight independent sums per thread: one chain of dependent additions per thread leaves the block waiting on one
  // load at a time (42 us for the 43,648 partial sums of d = 11.2 M; four sums of 256 threads 15, these 9); the order of
  // the additions is fixed
  constexpr int kSums = 8;
  double a[kSums] = {};
  int64_t k = threadIdx.x;
  for (; k + (kSums - 1) * kSumThreads < count; k += kSums * kSumThreads) {
#pragma unroll
    for (int q = 0; q < kSums; ++q) a[q] += partials[k + q * kSumThreads];
  }
#pragma unroll
  for (int q = 0; q < kSums; ++q)
    if (k + q * kSumThreads < count) a[q] += partials[k + q * kSumThreads];
#pragma unroll
  for (int o = kSums / 2; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < o; ++q) a[q] += a[q + o];
  const double t = block_sum<kSumThreads>(a[0]);
  if (threadIdx.x == 0) *out = t;
}

// Partial sums of detag_consensus_error_static: one slot per block of 256 columns.  The array is part of the
// library's code object, so every GPU the library runs on holds its own copy, at its own address, until the
// process ends.  In host code the name is only a handle for hipGetSymbolAddress; kernels receive the address
// that call returns.
__device__ __align__(256) double scratch[kStaticPartialsMax];

constexpr int kMaxDevices = 64;
double *g_scratch_ptr[kMaxDevices] = {};  // per device, set once by static_partials_init

}  // namespace

int static_partials_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hip_rc(hipErrorInvalidDevice);
  if (g_scratch_ptr[device]) return 0;
  double *ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch));
  if (e != hipSuccess) return hip_rc(e);
  g_scratch_ptr[device] = ptr;
  return 0;
}

double *static_partials(int device) {
  return device >= 0 && device < kMaxDevices ? g_scratch_ptr[device] : nullptr;
}

int launch_mean(const Shape &s, const void *X, float *xbar, void *stream) {
  const dim3 grid(ceil_div_i64(s.d, kThreads));
  auto st = static_cast<hipStream_t>(stream);
  auto go = [&](auto *kernel, auto *x) { kernel<<<grid, kThreads, 0, st>>>(s.n, s.d, s.ld, x, xbar); };
  const bool nt = fused::tile_access(s, s.bf16 ? 2 : 4, {X}) == kStream;
  if (s.bf16) go(nt ? &mean_kernel<bf16_t, true> : &mean_kernel<bf16_t, false>, static_cast<const bf16_t *>(X));
  else go(nt ? &mean_kernel<float, true> : &mean_kernel<float, false>, static_cast<const float *>(X));
  return hip_rc(hipGetLastError());
}

int64_t consensus_partials_count(const Shape &s) { return (s.d + kThreads - 1) / kThreads; }

int launch_consensus_error(const Shape &s, const void *X, double *partials, double *out, void *stream) {
  const int64_t blocks = consensus_partials_count(s);
  auto st = static_cast<hipStream_t>(stream);
  auto go = [&](auto *kernel, auto *x) { kernel<<<dim3(blocks), kThreads, 0, st>>>(s.n, s.d, s.ld, x, partials); };
  const bool nt = fused::tile_access(s, s.bf16 ? 2 : 4, {X}) == kStream;
  auto with = [&](auto *x) {
    using ST = std::remove_const_t<std::remove_pointer_t<decltype(x)>>;
    go(nt ? &consensus_partial_kernel<ST, true> : &consensus_partial_kernel<ST, false>, x);
  };
  if (s.bf16) with(static_cast<const bf16_t *>(X));
  else with(static_cast<const float *>(X));
  int rc = hip_rc(hipGetLastError());
  if (rc) return rc;
  sum_partials_kernel<<<1, kSumThreads, 0, st>>>(blocks, partials, out);
  return hip_rc(hipGetLastError());
}

}  // namespace detag
