// Gradient query and DeTAG phase in one pass, for the diagonal-quadratic
// objective on ring / 2-D torus gossip matrices:
//
//   G+ = h * (X - b) + sigma * z              (gradient query of Algorithm 2, at the phase-start model)
//   X+ = M(X - alpha*Y),  Y+ = M(Y + G+ - G)  (phase update, matrix form in the proof of Theorem 3)
// or, as Algorithm 2 prints it,  X+ = M(X) - alpha*M(Y),  Y+ = M(Y) + G+ - G
//
// with M the K-step accelerated gossip of Algorithm 3.  The gradient needs X,
// which the phase loads anyway, so fusing it saves one read of X, one write and
// one read of the gradient: per element the kernel reads X, Y, G, b and writes
// X, Y, G (28 B, fp32) where the two separate kernels move 36 B.  G is updated
// in place: row i of the old gradient is read just before the new one is stored.
//
// Same register-resident layout as the plain fused phase (one lane = one
// column, all n rows on chip; for 64 workers part of the tracker side waits in
// LDS, see kParkedRows).  The Gaussian noise is counter-based; one
// Philox block yields the four normals of four adjacent columns of one worker,
// so the four lanes of a quad each generate the block of one of four
// consecutive rows and exchange the results with two DPP quad permutes (a 4x4
// transpose): every lane evaluates one block per four rows instead of four.
#include "detag_internal.h"
#include "fused_common.hpp"
#include "noise_dev.hpp"

namespace detag {
namespace {

using namespace fused;

// Rows of the tracker side parked in LDS while the model side runs its rounds, for patterns of 64 workers.
// With all three arrays (u, v and the round scratch p) in registers a lane needs 192 + staging registers, two
// wavefronts per SIMD; with 48 of v's 64 rows in LDS (48 KiB per block, each lane reading back only what it
// wrote: no barrier) it needs 146, three wavefronts per SIMD and three blocks per compute unit, which hides
// more of the noise and round arithmetic under the other blocks' memory phases.
constexpr int kParkedRows = 48;
// HPW: the curvature h is an n x ld matrix (one row per worker, one more streamed array: 32 B per element) instead
// of one d-vector shared by all workers.
// Wavefronts per SIMD asked of the register allocator: three with the parked rows at 64 workers, else the phase
// kernels' figure, one less where all rows' loads of five arrays are in flight at once beside the three resident
// arrays (12 workers with per-worker curvature: 16 bytes of scratch per lane otherwise).
constexpr int quad_waves(int n, bool hpw) {
  return n >= 64 ? 3 : waves_per_simd(n, 1) - (hpw && n == 12 ? 1 : 0);
}

template <class T, typename ST, bool HPW, Access A>
__global__ __launch_bounds__(kThreads, quad_waves(T::n, HPW)) void fused_quadratic_kernel(
    ST *X, ST *Y, float *G, const float *__restrict__ h, const float *__restrict__ b, int64_t d, int64_t ld, Coef c,
    float alpha, int K, float sigma, uint32_t seed_lo, uint32_t seed_hi, uint32_t step) {
  constexpr int N = T::n;
  static_assert(N % 4 == 0, "rows are processed in groups of four");
  constexpr int NL = N >= 64 ? kParkedRows : 0;
  constexpr int NR = N - NL;
  constexpr int kAhead = kRowsAhead - (HPW && N >= 64 ? 2 : 0);  // two rows less of five arrays, or some of them spill
  constexpr int D = kAhead < N ? kAhead : N;
  __shared__ float vl[NL > 0 ? NL * kThreads : 1];
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  const uint32_t valid = uint32_t(d - tile < blockDim.x ? d - tile : blockDim.x);
  const uint32_t so = threadIdx.x * uint32_t(sizeof(ST)), fo = threadIdx.x * 4u;
  const unsigned j = threadIdx.x & 3u;
  const uint64_t q = uint64_t(tile + threadIdx.x) >> 2;
  const float hc = HPW ? 0.f : buf_load<float, A>(make_rsrc(h + tile, valid * 4u), fo);
  float u[N], p[N], vr[NR > 0 ? NR : 1];
  Loaded<ST> lx[N], ly[N];
  float lg[N], lb[N], lh[HPW ? N : 1];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
    ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
    lg[i] = buf_load<float, A>(row_of(G, tile, ld, i, valid), fo);
    lb[i] = buf_load<float, A>(row_of(b, tile, ld, i, valid), fo);
    if constexpr (HPW) lh[i] = buf_load<float, A>(row_of(h, tile, ld, i, valid), fo);
  }
  __builtin_amdgcn_sched_barrier(0);
  // All the noise of the tile is generated now, while the first rows' loads are in flight, and parked in p
  // (free until the rounds).  Generated inside the row loop instead, the Philox and Box-Muller arithmetic
  // spaces the loads out: fewer reads in flight, 2 % more kernel time on the 8x8 torus at d = 11.2 M.
  if (sigma != 0.f) {
#pragma unroll
    for (int i = 0; i < N; i += 4) {  // noise of rows i..i+3 at this lane's column
      float z[4];
      normal4(q, uint32_t(i) + j, step, seed_lo, seed_hi, z);
      quad_transpose(z, j);
      p[i] = z[0], p[i + 1] = z[1], p[i + 2] = z[2], p[i + 3] = z[3];
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = 0.f;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + D < N) {
      lx[i + D] = buf_request<ST, A>(row_of(X, tile, ld, i + D, valid), so);
      ly[i + D] = buf_request<ST, A>(row_of(Y, tile, ld, i + D, valid), so);
      lg[i + D] = buf_load<float, A>(row_of(G, tile, ld, i + D, valid), fo);
      lb[i + D] = buf_load<float, A>(row_of(b, tile, ld, i + D, valid), fo);
      if constexpr (HPW) lh[i + D] = buf_load<float, A>(row_of(h, tile, ld, i + D, valid), fo);
    }
    const float g = fmaf(sigma, p[i], (HPW ? lh[i] : hc) * (lx[i] - lb[i]));
    u[i] = fmaf(-alpha, ly[i], lx[i]);
    float vi = ly[i] + g - lg[i];
    pin_vgpr(vi);
    if (i < NR) vr[i] = vi;
    else vl[(i - NR) * kThreads + threadIdx.x] = vi;
    buf_store<float, A>(row_of(G, tile, ld, i, valid), fo, g);
    __builtin_amdgcn_sched_barrier(0);
  }
  ag_rounds<T>(u, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  X = launder_uniform(X);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, u[i]);
    if (i < NR) u[i] = vr[i];
    else u[i] = vl[(i - NR) * kThreads + threadIdx.x];
  }
  __builtin_amdgcn_sched_barrier(0);
  ag_rounds<T>(u, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  Y = launder_uniform(Y);
#pragma unroll
  for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, u[i]);
}

// Algorithm 2 as printed: the gossip runs on X and Y themselves and the gradients enter after it,
//   G+ = h*(X - b) + sigma*z;  X+ = M(X) - alpha*M(Y);  Y+ = M(Y) + G+ - G.
// The new gradient has to outlive both runs of rounds, so the tile keeps four values per element: X, Y and the
// round scratch in registers, the gradient in LDS (n KiB per block; every lane reads back only what it wrote, so
// there is no barrier).  The old gradient is read at the end, row by row just ahead of the row's stores, and
// overwritten in place: the same 28 B per element (32 B with per-worker curvature) as the ATC form.
template <class T, typename ST, bool HPW, Access A>
__global__ __launch_bounds__(kThreads, waves_per_simd(T::n, 1)) void fused_quadratic_alg2_kernel(
    ST *X, ST *Y, float *G, const float *__restrict__ h, const float *__restrict__ b, int64_t d, int64_t ld, Coef c,
    float alpha, int K, float sigma, uint32_t seed_lo, uint32_t seed_hi, uint32_t step) {
  constexpr int N = T::n;
  static_assert(N % 4 == 0, "rows are processed in groups of four");
  constexpr int D = kRowsAhead < N ? kRowsAhead : N;
  __shared__ float gl[N * kThreads];
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  const uint32_t valid = uint32_t(d - tile < blockDim.x ? d - tile : blockDim.x);
  const uint32_t so = threadIdx.x * uint32_t(sizeof(ST)), fo = threadIdx.x * 4u;
  const unsigned j = threadIdx.x & 3u;
  const uint64_t q = uint64_t(tile + threadIdx.x) >> 2;
  const float hc = HPW ? 0.f : buf_load<float, A>(make_rsrc(h + tile, valid * 4u), fo);
  float u[N], v[N], p[N];
  {
    Loaded<ST> lx[N], ly[N];
    float lb[N], lh[HPW ? N : 1];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
      ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
      lb[i] = buf_load<float, A>(row_of(b, tile, ld, i, valid), fo);
      if constexpr (HPW) lh[i] = buf_load<float, A>(row_of(h, tile, ld, i, valid), fo);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (sigma != 0.f) {  // the tile's noise, generated while the first rows' loads are in flight
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        float z[4];
        normal4(q, uint32_t(i) + j, step, seed_lo, seed_hi, z);
        quad_transpose(z, j);
        p[i] = z[0], p[i + 1] = z[1], p[i + 2] = z[2], p[i + 3] = z[3];
      }
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) p[i] = 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (i + D < N) {
        lx[i + D] = buf_request<ST, A>(row_of(X, tile, ld, i + D, valid), so);
        ly[i + D] = buf_request<ST, A>(row_of(Y, tile, ld, i + D, valid), so);
        lb[i + D] = buf_load<float, A>(row_of(b, tile, ld, i + D, valid), fo);
        if constexpr (HPW) lh[i + D] = buf_load<float, A>(row_of(h, tile, ld, i + D, valid), fo);
      }
      gl[i * kThreads + threadIdx.x] = fmaf(sigma, p[i], (HPW ? lh[i] : hc) * (lx[i] - lb[i]));
      u[i] = lx[i];
      v[i] = ly[i];
      pin_vgpr(v[i]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  ag_rounds<T>(v, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  ag_rounds<T>(u, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  X = launder_uniform(X), Y = launder_uniform(Y);
  float lgo[N];
#pragma unroll
  for (int i = 0; i < D; ++i) lgo[i] = buf_load<float, A>(row_of(G, tile, ld, i, valid), fo);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + D < N) lgo[i + D] = buf_load<float, A>(row_of(G, tile, ld, i + D, valid), fo);
    const float g = gl[i * kThreads + threadIdx.x];
    buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, fmaf(-alpha, v[i], u[i]));
    buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, v[i] + g - lgo[i]);
    buf_store<float, A>(row_of(G, tile, ld, i, valid), fo, g);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Both forms for small calls: two wavefronts to a block on the same 64 columns, the first with the model side, the second with
// the tracker side, whose rounds so run beside each other.  ATC: both read X and Y, the tracker side takes the gradient query.
// Algorithm 2 as printed: the model side, which reads X, takes it and hands the gradient over in LDS, as the tracker side does
// with the gossiped tracker.  Nothing that both read is stored before the barrier.  Same arithmetic as the kernels above, same
// bits.
template <class T, typename ST, bool HPW, bool ALG2>
__global__ __launch_bounds__(kPairThreads, 2) void fused_quadratic_pair_kernel(
    ST *X, ST *Y, float *G, const float *__restrict__ h, const float *__restrict__ b, int64_t d, int64_t ld, Coef c,
    float alpha, int K, float sigma, uint32_t seed_lo, uint32_t seed_hi, uint32_t step) {
  constexpr int N = T::n;
  constexpr int D = kRowsAhead < N ? kRowsAhead : N;
  constexpr Access A = kKeep;
  constexpr int kQuerySide = ALG2 ? 0 : 1;
  __shared__ float tracker[ALG2 ? N * 64 : 1], gradient[ALG2 ? N * 64 : 1];
  const int side = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * 64;
  const uint32_t valid = uint32_t(d - tile < 64 ? d - tile : 64);
  const uint32_t so = lane * uint32_t(sizeof(ST)), fo = lane * 4u;
  float z[N], p[N];
  if (side == kQuerySide) {
    const unsigned j = lane & 3u;
    const uint64_t q = uint64_t(tile + lane) >> 2;
    const float hc = HPW ? 0.f : buf_load<float, A>(make_rsrc(h + tile, valid * 4u), fo);
    Loaded<ST> lx[N], ly[N];
    float lg[N], lb[N], lh[HPW ? N : 1];
    auto request = [&](int i) {
      lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
      lb[i] = buf_load<float, A>(row_of(b, tile, ld, i, valid), fo);
      if constexpr (HPW) lh[i] = buf_load<float, A>(row_of(h, tile, ld, i, valid), fo);
      if constexpr (!ALG2) {
        ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
        lg[i] = buf_load<float, A>(row_of(G, tile, ld, i, valid), fo);
      }
    };
#pragma unroll
    for (int i = 0; i < D; ++i) request(i);
    __builtin_amdgcn_sched_barrier(0);
    if (sigma != 0.f) {  // under the first rows' loads
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        float r[4];
        normal4(q, uint32_t(i) + j, step, seed_lo, seed_hi, r);
        quad_transpose(r, j);
        p[i] = r[0], p[i + 1] = r[1], p[i + 2] = r[2], p[i + 3] = r[3];
      }
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) p[i] = 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (i + D < N) request(i + D);
      const float g = fmaf(sigma, p[i], (HPW ? lh[i] : hc) * (lx[i] - lb[i]));
      if constexpr (ALG2) {
        gradient[i * 64 + lane] = g;
        z[i] = lx[i];
      } else {
        z[i] = ly[i] + g - lg[i];
        pin_vgpr(z[i]);
        buf_store<float, A>(row_of(G, tile, ld, i, valid), fo, g);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    Loaded<ST> lz[N], ly[N];
#pragma unroll
    for (int i = 0; i < N; ++i) lz[i] = buf_request<ST, A>(row_of(ALG2 ? Y : X, tile, ld, i, valid), so);
    if constexpr (ALG2) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i) z[i] = lz[i];
    } else {
#pragma unroll
      for (int i = 0; i < D; ++i) ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i + D < N) ly[i + D] = buf_request<ST, A>(row_of(Y, tile, ld, i + D, valid), so);
        z[i] = fmaf(-alpha, ly[i], lz[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  ag_rounds<T>(z, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!ALG2) {
    __syncthreads();
    ST *Z = side ? Y : X;
#pragma unroll
    for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(Z, tile, ld, i, valid), so, z[i]);
  } else {
    float lg[N];
    if (side) {
#pragma unroll
      for (int i = 0; i < D; ++i) lg[i] = buf_load<float, A>(row_of(G, tile, ld, i, valid), fo);
#pragma unroll
      for (int i = 0; i < N; ++i) tracker[i * 64 + lane] = z[i];
    }
    __syncthreads();
    if (side == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, fmaf(-alpha, tracker[i * 64 + lane], z[i]));
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i + D < N) lg[i + D] = buf_load<float, A>(row_of(G, tile, ld, i + D, valid), fo);
        const float g = gradient[i * 64 + lane];
        buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, z[i] + g - lg[i]);
        buf_store<float, A>(row_of(G, tile, ld, i, valid), fo, g);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

template <class T>
int launch_s(const Shape &s, bool alg2, void *X, void *Y, float *G, const float *h, bool hpw, const float *b,
             const Coef &c, float alpha, int K, float sigma, uint64_t seed, uint32_t step, void *stream) {
  const bool pair = pair_serves(s.d, K, true);
  const int threads = pair ? kPairThreads : kThreads;
  const dim3 grid(ceil_div_i64(s.d, pair ? 64 : kThreads));
  auto st = static_cast<hipStream_t>(stream);
  const uint32_t slo = uint32_t(seed & 0xffffffffu), shi = uint32_t(seed >> 32);
  auto go = [&](auto *kernel, auto *x) {
    kernel<<<grid, threads, 0, st>>>(x, static_cast<decltype(x)>(Y), G, h, b, s.d, s.ld, c, alpha, K, sigma, slo, shi, step);
  };
  auto with = [&](auto access, auto per_worker, auto *x) {
    using ST = std::remove_pointer_t<decltype(x)>;
    if (alg2) go(&fused_quadratic_alg2_kernel<T, ST, per_worker, access>, x);
    else go(&fused_quadratic_kernel<T, ST, per_worker, access>, x);
  };
  auto with_h = [&](auto access, auto *x) { hpw ? with(access, std::true_type{}, x) : with(access, std::false_type{}, x); };
  if (pair) {
    auto with_pair = [&](auto *x) {
      using ST = std::remove_pointer_t<decltype(x)>;
      auto form = [&](auto per_worker) {
        alg2 ? go(&fused_quadratic_pair_kernel<T, ST, per_worker, true>, x) : go(&fused_quadratic_pair_kernel<T, ST, per_worker, false>, x);
      };
      hpw ? form(std::true_type{}) : form(std::false_type{});
    };
    if (s.bf16) with_pair(static_cast<bf16_t *>(X));
    else with_pair(static_cast<float *>(X));
    return hip_rc(hipGetLastError());
  }
  const int per_element = (s.bf16 ? 4 : 8) + 8 + (hpw ? 4 : 0);
  auto with_type = [&](auto access) {
    if (s.bf16) with_h(access, static_cast<bf16_t *>(X));
    else with_h(access, static_cast<float *>(X));
  };
  const uint64_t line = register_line(s, per_element, alg2 ? kAlg2Form : kAtcForm);
  if (tile_access(s, per_element, {X, Y, G, hpw ? h : nullptr, b}, line) == kStream) with_type(AccessTag<kStream>{});
  else with_type(AccessTag<kKeep>{});
  return hip_rc(hipGetLastError());
}

}  // namespace

int launch_fused_quadratic(const Shape &s, const HostW &W, bool alg2, void *X, void *Y, float *G, const float *h,
                           bool h_per_worker, const float *b, float alpha, int K, float eta, float sigma, uint64_t seed,
                           uint32_t step, void *stream) {
  if (K < 1) return -1;
  const Coef c = make_coef(W, eta);
  return with_pattern(W, [&](auto t) {
    return launch_s<decltype(t)>(s, alg2, X, Y, G, h, h_per_worker, b, c, alpha, K, sigma, seed, step, stream);
  });
}

}  // namespace detag
