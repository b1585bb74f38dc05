// K-round fused DeTAG phase for ring and 2-D torus gossip matrices.
//
// Gossip mixes workers (rows) and never columns, so a set of columns together
// with ALL n rows is a closed system: one lane owns one column, keeps the n
// worker values of that column in registers, and runs all K rounds of
// Algorithm 3 there.  The neighbour pattern is a compile-time function of the
// row index, so every z[j] below is a fixed register.  HBM sees each state
// element once on the way in and once on the way out, whatever K is:
//   phase (ATC/ALG2): read X, Y, Gnew, Gold, write X, Y  = 24 B per element (fp32 state)
//   gossip only     : read Z, write Z                    =  8 B per element
// A wavefront reads 256 contiguous bytes of one row per load instruction and a
// 256-thread block 1 KiB; rows are n*ld apart, which the hardware sees as n
// (times four matrices) sequential streams.
//
// Paper: Algorithm 3 (accelerated gossip), Algorithm 2 (phase update) and the
// matrix form in the proof of Theorem 3.
#include "detag_internal.h"
#include "fused_common.hpp"

namespace detag {
namespace {

using namespace fused;


// MODE 0: Z <- M(Z) on X.  MODE 1 (ATC): X <- M(X - alpha*Y), Y <- M(Y + Gn - Go).
// MODE 2 (ALG2): X <- M(X) - alpha*M(Y), Y <- M(Y) + Gn - Go.
// MODE 3 (D-PSGD baseline of the Experiments section): X <- W^T X - alpha*Gn, one plain round (c built with eta = 0).
template <class T, typename ST, int MODE, Access A>
__global__ __launch_bounds__(kThreads, waves_per_simd(T::n, MODE)) void fused_structured_kernel(
    ST *X, ST *Y, const float *__restrict__ Gn, const float *__restrict__ Go, int64_t d, int64_t ld, Coef c,
    float alpha, int K) {
  constexpr int N = T::n;
  constexpr int D = kRowsAhead < N ? kRowsAhead : N;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  const uint32_t valid = uint32_t(d - tile < blockDim.x ? d - tile : blockDim.x);
  const uint32_t so = threadIdx.x * uint32_t(sizeof(ST));  // lane byte offset in a state row
  const uint32_t go4 = threadIdx.x * 4u;                   // ... in an fp32 row
  float u[N], p[N];
  if constexpr (MODE == 0) {
    Loaded<ST> lx[N];
#pragma unroll
    for (int i = 0; i < N; ++i) lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = lx[i];
    ag_rounds<T>(u, p, c, K);
    __builtin_amdgcn_sched_barrier(0);
    X = launder_uniform(X);
#pragma unroll
    for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, u[i]);
  } else if constexpr (MODE == 3) {
    Loaded<ST> lx[N];
#pragma unroll
    for (int i = 0; i < N; ++i) lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
    __builtin_amdgcn_sched_barrier(0);
    X = launder_uniform(X);
    float lg[N];  // gradient rows arrive a few rows ahead of the stores that consume them
#pragma unroll
    for (int i = 0; i < D; ++i) lg[i] = buf_load<float, A>(row_of(Gn, tile, ld, i, valid), go4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = lx[i];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (i + D < N) lg[i + D] = buf_load<float, A>(row_of(Gn, tile, ld, i + D, valid), go4);
      buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, fmaf(-alpha, lg[i], fmaf(c.b, lap<T>(u, i), u[i])));
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    static_assert(MODE == 1 || MODE == 2, "unknown mode");
    float v[N];
    if constexpr (MODE == 1) {
      Loaded<ST> lx[N], ly[N];
      float lgn[N], lgo[N];
#pragma unroll
      for (int i = 0; i < D; ++i) {
        lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
        ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
        lgn[i] = buf_load<float, A>(row_of(Gn, tile, ld, i, valid), go4);
        lgo[i] = buf_load<float, A>(row_of(Go, tile, ld, i, valid), go4);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i + D < N) {
          lx[i + D] = buf_request<ST, A>(row_of(X, tile, ld, i + D, valid), so);
          ly[i + D] = buf_request<ST, A>(row_of(Y, tile, ld, i + D, valid), so);
          lgn[i + D] = buf_load<float, A>(row_of(Gn, tile, ld, i + D, valid), go4);
          lgo[i + D] = buf_load<float, A>(row_of(Go, tile, ld, i + D, valid), go4);
        }
        u[i] = fmaf(-alpha, ly[i], lx[i]);
        v[i] = ly[i] + lgn[i] - lgo[i];
        pin_vgpr(v[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
      ag_rounds<T>(u, p, c, K);
      __builtin_amdgcn_sched_barrier(0);
      X = launder_uniform(X);
#pragma unroll
      for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, u[i]);
      __builtin_amdgcn_sched_barrier(0);
      ag_rounds<T>(v, p, c, K);
      __builtin_amdgcn_sched_barrier(0);
      Y = launder_uniform(Y);
#pragma unroll
      for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, v[i]);
    } else {
      Loaded<ST> lx[N], ly[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        lx[i] = buf_request<ST, A>(row_of(X, tile, ld, i, valid), so);
        ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        u[i] = lx[i], v[i] = ly[i];
        // bf16: or its load moves behind the tracker's rounds; fp32 rows may arrive under them (waited for ahead of them, torus
        // 8x8, d = 312,500, K = 12 117 and 125 us, K = 4 the same)
        if constexpr (sizeof(ST) == 2) pin_vgpr(u[i]);
      }
      ag_rounds<T>(v, p, c, K);
      __builtin_amdgcn_sched_barrier(0);
      ag_rounds<T>(u, p, c, K);
      __builtin_amdgcn_sched_barrier(0);
      // p is free now: the gradient rows are fetched a few rows ahead of the stores
      X = launder_uniform(X), Y = launder_uniform(Y);
      float lgn[N], lgo[N];
#pragma unroll
      for (int i = 0; i < D; ++i) {
        lgn[i] = buf_load<float, A>(row_of(Gn, tile, ld, i, valid), go4);
        lgo[i] = buf_load<float, A>(row_of(Go, tile, ld, i, valid), go4);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i + D < N) {
          lgn[i + D] = buf_load<float, A>(row_of(Gn, tile, ld, i + D, valid), go4);
          lgo[i + D] = buf_load<float, A>(row_of(Go, tile, ld, i + D, valid), go4);
        }
        buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, fmaf(-alpha, v[i], u[i]));
        buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, v[i] + lgn[i] - lgo[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// The phase for small calls: a block is two wavefronts on the same 64 columns, the first with the model side (X), the second
// with the tracker side (Y), so that their rounds run beside each other and not one after the other.  Both read Y (the second
// time from the caches); nothing is stored before the barrier behind both sides' loads.  MODE 2 hands the gossiped tracker to
// the model side through LDS.  Same arithmetic as the kernel above, same bits.
template <class T, typename ST, int MODE>
__global__ __launch_bounds__(kPairThreads, 2) void fused_pair_kernel(
    ST *X, ST *Y, const float *__restrict__ Gn, const float *__restrict__ Go, int64_t d, int64_t ld, Coef c, float alpha, int K) {
  constexpr int N = T::n;
  constexpr int D = kRowsAhead < N ? kRowsAhead : N;
  constexpr Access A = kKeep;
  __shared__ float handed[MODE == 2 ? N * 64 : 1];
  const int side = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * 64;
  const uint32_t valid = uint32_t(d - tile < 64 ? d - tile : 64);
  const uint32_t so = lane * uint32_t(sizeof(ST)), fo = lane * 4u;
  float z[N], p[N];
  if (MODE == 2 || side == 0) {
    const ST *Z = MODE == 2 && side ? Y : X;
    Loaded<ST> lz[N], ly[N];
#pragma unroll
    for (int i = 0; i < N; ++i) lz[i] = buf_request<ST, A>(row_of(Z, tile, ld, i, valid), so);
    if constexpr (MODE == 2) {
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
  } else {
    Loaded<ST> ly[N];
    float lgn[N], lgo[N];
#pragma unroll
    for (int i = 0; i < D; ++i) {
      ly[i] = buf_request<ST, A>(row_of(Y, tile, ld, i, valid), so);
      lgn[i] = buf_load<float, A>(row_of(Gn, tile, ld, i, valid), fo);
      lgo[i] = buf_load<float, A>(row_of(Go, tile, ld, i, valid), fo);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (i + D < N) {
        ly[i + D] = buf_request<ST, A>(row_of(Y, tile, ld, i + D, valid), so);
        lgn[i + D] = buf_load<float, A>(row_of(Gn, tile, ld, i + D, valid), fo);
        lgo[i + D] = buf_load<float, A>(row_of(Go, tile, ld, i + D, valid), fo);
      }
      z[i] = ly[i] + lgn[i] - lgo[i];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  ag_rounds<T>(z, p, c, K);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (MODE == 1) {
    __syncthreads();
    ST *Z = side ? Y : X;
#pragma unroll
    for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(Z, tile, ld, i, valid), so, z[i]);
  } else {
    float lgn[N], lgo[N];
    if (side) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        lgn[i] = buf_load<float, A>(row_of(Gn, tile, ld, i, valid), fo);
        lgo[i] = buf_load<float, A>(row_of(Go, tile, ld, i, valid), fo);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) handed[i * 64 + lane] = z[i];
    }
    __syncthreads();
    if (side == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(X, tile, ld, i, valid), so, fmaf(-alpha, handed[i * 64 + lane], z[i]));
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i + D < N) {
          lgn[i + D] = buf_load<float, A>(row_of(Gn, tile, ld, i + D, valid), fo);
          lgo[i + D] = buf_load<float, A>(row_of(Go, tile, ld, i + D, valid), fo);
        }
        buf_store<ST, A>(row_of(Y, tile, ld, i, valid), so, z[i] + lgn[i] - lgo[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// z_{r+1} of worker i from the rows of z_r and its own z_{r-1}: what a round given z_{r-1} computes, alone or among others.
template <class T>
__device__ __forceinline__ float next_iterate(const float (&z)[T::n], int i, float prev, const Coef &c) {
  return z[i] + fmaf(c.eta, z[i] - prev, c.b * lap<T>(z, i));
}

// One round of Algorithm 3 with z_{r-1} given (one iteration of Algorithm 2's communication), for the patterns above:
//   out = z_r + b * sum_nb (z_j - z_i) + eta * (z_r - z_{r-1}),   b = (1+eta) * w_nb.
// All n rows of z_r in registers, z_{r-1} streamed a few rows ahead of the stores: 12 B per element (fp32), every row
// read once.  Every row of z_r is in registers before the first store and a row of z_{r-1} is read before the same
// row of out is written, so out may be z_{r-1} (the caller's usual choice) or z_r itself.
template <class T, typename ST, Access A>
__global__ __launch_bounds__(kThreads, waves_per_simd(T::n, 0)) void structured_round_kernel(
    const ST *cur, const ST *prev, ST *out, int64_t d, int64_t ld, Coef c) {
  constexpr int N = T::n;
  constexpr int D = kRowsAhead < N ? kRowsAhead : N;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  const uint32_t valid = uint32_t(d - tile < blockDim.x ? d - tile : blockDim.x);
  const uint32_t so = threadIdx.x * uint32_t(sizeof(ST));
  float u[N];
  Loaded<ST> lc[N], lp[N];
#pragma unroll
  for (int i = 0; i < N; ++i) lc[i] = buf_request<ST, A>(row_of(cur, tile, ld, i, valid), so);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < D; ++i) lp[i] = buf_request<ST, A>(row_of(prev, tile, ld, i, valid), so);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) u[i] = lc[i];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + D < N) lp[i + D] = buf_request<ST, A>(row_of(prev, tile, ld, i + D, valid), so);
    buf_store<ST, A>(row_of(out, tile, ld, i, valid), so, next_iterate<T>(u, i, lp[i], c));
    __builtin_amdgcn_sched_barrier(0);
  }
}

// What a stored state holds of a value.
template <typename ST>
__device__ __forceinline__ float as_stored(float v) { return to_f32(from_f32<ST>(v)); }

// K rounds of the kernel above with z_{-1} = z_0 in one launch, in place and with its bits (bf16 state is rounded after every
// round): z_r and z_{r-1} of all workers stay in registers, a round writes over z_{r-1}.  8 B per element whatever K, where a
// launch per round moves 12 each time.  blockIdx.y picks the matrix: the model replica and the tracker of a phase take one
// launch.  A phase of Algorithm 2 on a ring of 16, d = 272,474, R = 6, its twelve rounds on a stream beside the gradient
// queries: 245 us with a launch per round, 177 so.
template <class T, typename ST, Access A>
__global__ __launch_bounds__(kThreads, waves_per_simd(T::n, 0)) void structured_rounds_kernel(ST *Z0, ST *Z1, int64_t d,
                                                                                           int64_t ld, Coef c, int K) {
  constexpr int N = T::n;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  const uint32_t valid = uint32_t(d - tile < blockDim.x ? d - tile : blockDim.x);
  const uint32_t so = threadIdx.x * uint32_t(sizeof(ST));
  ST *Z = blockIdx.y ? Z1 : Z0;
  float z[N], p[N];
  Loaded<ST> lz[N];
#pragma unroll
  for (int i = 0; i < N; ++i) lz[i] = buf_request<ST, A>(row_of(Z, tile, ld, i, valid), so);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) p[i] = z[i] = lz[i];
  for (int r = 0; r + 1 < K; r += 2) {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = as_stored<ST>(next_iterate<T>(z, i, p[i], c));
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = as_stored<ST>(next_iterate<T>(p, i, z[i], c));
  }
  if (K & 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = next_iterate<T>(z, i, p[i], c);
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = p[i];
  }
  __builtin_amdgcn_sched_barrier(0);
  Z = launder_uniform(Z);
#pragma unroll
  for (int i = 0; i < N; ++i) buf_store<ST, A>(row_of(Z, tile, ld, i, valid), so, z[i]);
}

template <class T, typename ST, Access A>
int launch_t(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, const Coef &c,
             float alpha, int K, void *stream) {
  const int threads = block_threads(s.d);
  const dim3 grid(ceil_div_i64(s.d, threads));
  auto st = static_cast<hipStream_t>(stream);
  auto go = [&](auto *kernel) {
    kernel<<<grid, threads, 0, st>>>(static_cast<ST *>(X), static_cast<ST *>(Y), Gn, Go, s.d, s.ld, c, alpha, K);
  };
  switch (mode) {
    case 0: go(&fused_structured_kernel<T, ST, 0, A>); break;
    case 1: go(&fused_structured_kernel<T, ST, 1, A>); break;
    case 3: go(&fused_structured_kernel<T, ST, 3, A>); break;
    default: go(&fused_structured_kernel<T, ST, 2, A>); break;
  }
  return hip_rc(hipGetLastError());
}

template <class T>
int launch_s(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, const Coef &c,
             float alpha, int K, void *stream) {
  if ((mode == 1 || mode == 2) && pair_serves(s.d, K, false)) {
    const dim3 grid(ceil_div_i64(s.d, 64));
    auto pair = [&](auto *kernel, auto of) {
      using ST = decltype(of);
      kernel<<<grid, kPairThreads, 0, static_cast<hipStream_t>(stream)>>>(static_cast<ST *>(X), static_cast<ST *>(Y), Gn, Go, s.d,
                                                                          s.ld, c, alpha, K);
      return hip_rc(hipGetLastError());
    };
    if (s.bf16) return mode == 1 ? pair(&fused_pair_kernel<T, bf16_t, 1>, bf16_t{}) : pair(&fused_pair_kernel<T, bf16_t, 2>, bf16_t{});
    return mode == 1 ? pair(&fused_pair_kernel<T, float, 1>, 0.f) : pair(&fused_pair_kernel<T, float, 2>, 0.f);
  }
  const int state = s.bf16 ? 2 : 4, per_element = mode == 0 ? state : mode == 3 ? state + 4 : 2 * state + 8;
  auto go = [&](auto access) {
    return s.bf16 ? launch_t<T, bf16_t, access>(s, mode, X, Y, Gn, Go, c, alpha, K, stream)
                  : launch_t<T, float, access>(s, mode, X, Y, Gn, Go, c, alpha, K, stream);
  };
  static_assert(kGossipForm == 0 && kAtcForm == 1 && kAlg2Form == 2 && kDpsgdForm == 3, "the modes in order");
  const uint64_t line = register_line(s, per_element, Form(mode));
  return tile_access(s, per_element, {X, Y, Gn, Go}, line) == kStream ? go(AccessTag<kStream>{}) : go(AccessTag<kKeep>{});
}

}  // namespace

bool fused_structured_available(const HostW &W) {
  return with_pattern(W, [](auto) { return 0; }) == 0;
}

int launch_fused_structured(const Shape &s, const HostW &W, int mode, void *X, void *Y, const float *Gn,
                            const float *Go, float alpha, int K, float eta, void *stream) {
  if (K < 1) return -1;
  const Coef c = make_coef(W, eta);
  return with_pattern(W, [&](auto t) { return launch_s<decltype(t)>(s, mode, X, Y, Gn, Go, c, alpha, K, stream); });
}

int launch_structured_round(const Shape &s, const HostW &W, const void *cur, const void *prev, void *out, float eta,
                            void *stream) {
  const Coef c = make_coef(W, eta);
  const int threads = block_threads(s.d);
  const dim3 grid(ceil_div_i64(s.d, threads));
  auto st = static_cast<hipStream_t>(stream);
  return with_pattern(W, [&](auto t) {
    using T = decltype(t);
    auto go = [&](auto *kernel, auto of) {
      using ST = decltype(of);
      kernel<<<grid, threads, 0, st>>>(static_cast<const ST *>(cur), static_cast<const ST *>(prev), static_cast<ST *>(out), s.d,
                                       s.ld, c);
    };
    auto with = [&](auto access) {
      if (s.bf16) go(&structured_round_kernel<T, bf16_t, access>, bf16_t{});
      else go(&structured_round_kernel<T, float, access>, float{});
      return hip_rc(hipGetLastError());
    };
    const int per_element = 3 * (s.bf16 ? 2 : 4);
    const Access access = tile_access(s, per_element, {cur, prev, out}, register_line(s, per_element, kRoundForm));
    return access == kStream ? with(AccessTag<kStream>{}) : with(AccessTag<kKeep>{});
  });
}

int launch_structured_rounds(const Shape &s, const HostW &W, void *Z0, void *Z1, int K, float eta, void *stream) {
  const Coef c = make_coef(W, eta);
  const int threads = block_threads(s.d);
  const dim3 grid(ceil_div_i64(s.d, threads), Z1 ? 2 : 1);
  auto st = static_cast<hipStream_t>(stream);
  return with_pattern(W, [&](auto t) {
    using T = decltype(t);
    auto go = [&](auto *kernel, auto of) {
      using ST = decltype(of);
      kernel<<<grid, threads, 0, st>>>(static_cast<ST *>(Z0), static_cast<ST *>(Z1), s.d, s.ld, c, K);
    };
    auto with = [&](auto access) {
      if (s.bf16) go(&structured_rounds_kernel<T, bf16_t, access>, bf16_t{});
      else go(&structured_rounds_kernel<T, float, access>, float{});
      return hip_rc(hipGetLastError());
    };
    const int per_element = (Z1 ? 2 : 1) * (s.bf16 ? 2 : 4);
    const Access access = tile_access(s, per_element, {Z0, Z1}, register_line(s, per_element, kGossipForm));
    return access == kStream ? with(AccessTag<kStream>{}) : with(AccessTag<kKeep>{});
  });
}

}  // namespace detag
