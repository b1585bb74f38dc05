// Shared by the register-resident fused kernels: the compile-time neighbour
// patterns (ring, 2-D torus) and K rounds of Algorithm 3 on a column held in
// registers.
#pragma once

#include <initializer_list>
#include <type_traits>

#include "detag_internal.h"
#include "dev_common.hpp"

namespace detag {
namespace fused {

constexpr int kThreads = 256;

// Threads of a block.  No two wavefronts of a block work together, so its size only decides how columns spread over the
// chip: up to 32,768 columns make 128 blocks of 256 threads or fewer and take one wavefront per block, which spreads them
// over all compute units (rounds of 4 to 64 workers 1 to 5 % faster at 8,192 to 32,768 columns).  Beyond, both sizes are
// within 2 %.  Phases of so few columns take the kernels of pair_serves.
inline int block_threads(int64_t d) { return d <= 32768 ? 64 : kThreads; }

// Small calls run the model side and the tracker side of a phase in two wavefronts of a block (fused_pair_kernel,
// fused_quadratic_pair_kernel), which halves the chain of rounds where there are too few columns to fill the chip; with more,
// the second read of a matrix costs more than that saves.  One wavefront for both sides and two, K = 8, fp32 (bf16 within 5 %
// of it), replayed from a recorded graph: phase, torus 8x8 d = 1,000 15.4 and 9.2 us, 32,000 19.6 and 15.3, 65,000 26.1 and
// 22.5, 130,000 41.2 and 50.6; ring of 32 6.7 and 4.5, 8.8 and 7.5, 12.8 and 11.7, 18.3 and 17.7; fused step, torus 8x8 19.6
// and 13.7, 22.7 and 16.9, at 45,000 25.1 and 18.8, at 65,000 28.8 and 24.8; ring of 16 at 60,000 7.5 and 7.8; Algorithm 2 as
// printed gains more.  K = 1: phase, ring of 32, d = 5,001 3.9 and 3.1, 32,000 5.5 and 5.5, 45,000 7.3 and 7.5.  Three states in
// turn: K = 1, step, torus 8x8 24,000 12.5 and 11.9, 32,000 13.9 and 12.4, ring of 32 32,000 7.6 and 7.7; K = 2 and 3, phase, ring
// of 16 48,000 4.7 and 4.7, 5.0 and 4.8, 65,000 6.0 and 6.0, 6.2 and 6.2, step 5.7 and 5.7, 6.1 and 5.9, 65,000 6.5 and 7.1, 6.7
// and 7.2; bf16 gains a little more.
constexpr int kPairThreads = 128;
inline bool pair_serves(int64_t d, int K, bool with_query) {
  return d <= (K == 1 ? 32768 : K >= 4 && !with_query ? 65536 : 49152);
}

// Workgroups are handed to the eight XCDs (each with its own L2) round-robin by their index.  Mapping index b
// to column tile (b % 8) * (tiles / 8) + b / 8 gives every XCD one contiguous eighth of the columns instead of
// every eighth tile, so the lines one L2 holds are neighbours in memory.  The tiles past a multiple of eight
// keep their own index.
__device__ __forceinline__ int64_t xcd_tile(uint32_t b, uint32_t tiles) {
  const uint32_t per = tiles / 8u;
  return b < per * 8u ? int64_t(b % 8u) * per + b / 8u : int64_t(b);
}

// Whether column tiles share cache lines of 128 bytes: rows that do not start on one (an odd pitch, a shifted base).
inline bool shares_lines(const Shape &s, std::initializer_list<const void *> matrices, uint64_t line = 128) {
  uint64_t starts = uint64_t(s.ld) * (s.bf16 ? 2 : 4);
  for (const void *p : matrices) starts |= reinterpret_cast<uint64_t>(p);
  return starts % line != 0;
}
// What the matrices of a call that walks column tiles take together.
inline int64_t footprint(const Shape &s, int per_element) { return int64_t(s.n) * s.ld * per_element; }

// Whether the loads of a kernel that walks rows as they lie stream past the caches (its stores do in any case).  Up to
// 128 MiB they find their matrices in the memory-side cache, three states in turn as well: phase end of 64 x 100,001
// (122 MiB, fp32) 38.9 -> 34.2 us, gradient of 16 x 272,474 12.3 -> 11.2, accumulation 11.4 -> 10.4; at 200 MiB all of them
// but the gradient with one curvature per worker are slower so.  The updates of tracker and model and the accumulation, which
// read what they write and little else, up to 104 MiB (16 workers, streamed and kept: tracker 104 MiB 24.3 and 24.2, 126 MiB
// 29.3 and 31.1; with the model 28.4 and 27.8, 33.5 and 35.6; accumulation 27.4 and 27.2, 32.7 and 34.5; phase end 31.1 and
// 27.4, 38.0 and 34.5).
constexpr int kRowLoadsMiB = 128, kUpdateLoadsMiB = 104;
inline bool loads_stream(const Shape &s, int per_element, int up_to_mib = kRowLoadsMiB) {
  return footprint(s, per_element) > (int64_t(up_to_mib) << 20);
}

// How the register-resident kernels and those with one launch per round treat the caches.
// Small calls leave their matrices to the caches.  The memory-side cache holds 256 MB and a program has other matrices too:
// up to 80 MiB a call's matrices stay, where the next call finds them (gradient-fused step, ring of 16: d = 272,474 (70 MB)
// 22 -> 19 us, three states in turn as well; a state that no call has touched lately gains half of that).  Measured at 85,
// 95, 105, 115 and 128 MiB over all calls of ring 16 and torus 8x8: with one state the caches stay 5 to 15 % ahead; with
// three in turn -11 to +6 % up to 105 MiB, from 115 on 5 to 20 % behind.  So the line lies below where it can lose.
// Beyond, a call streams, but only if its tiles have their cache lines to themselves: a shared line that streams is gone
// before the other tile wants it, or goes to memory half written.  Streamed and kept, fp32, pitch 1,000,003, K = 4: phase,
// torus 8x8 388 and 296 us, one round 165 and 145, gradient-fused step 465 and 364; ring of 16, pitch 600,001 52 and 50, 65
// and 60.  On lines streaming is 2 to 10 % ahead.
// A kernel may set another mark than the line: rows that start on a multiple of `line` bytes stream.
inline Access tile_access(const Shape &s, int per_element, std::initializer_list<const void *> matrices, uint64_t line = 128) {
  return footprint(s, per_element) > (int64_t(80) << 20) && !shares_lines(s, matrices, line) ? kStream : kKeep;
}

// The mark of the register-resident kernels.  Few rows share few lines, and a row of bf16 state that starts on half a line
// shares with one neighbour.  Streamed and kept, bf16 rows on half lines: the ATC phase and the step fused with it (torus
// 8x8, 183 MiB 54.0 and 59.7 us, fused step 68 and 73, 732 MiB 212 and 213, 275 and 281; ring of 4, 183 MiB 45.8 and 49.9, 732
// MiB 196 and 197; rings of 16 and 32, 183 MiB 50.1 and 52.6, 50.5 and 53.8, but 732 MiB 206 and 200, 208 and 203, fused step
// 273 and 257, 271 and 261); Algorithm 2's phase, ring of
// 4, 220 MiB a call 63 and 67, 800 MiB 209 and 213, ring of 16 100 MiB 29 and 27, 220 MiB 61 and 64, 300 MiB 91 and 86; the
// D-PSGD step, ring of 16, 220 MiB 60 and 63, 800 MiB 220 and 218; plain gossip, ring of 8, 100 MiB 44 and 44, 400 MiB 169 and
// 175, ring of 16 181 and 174; one round, ring of 8, 100 MiB 21 and 24, torus 8x8, 140 MiB 31 and 33, 300 MiB 69 and 67.
// Wherever the rows start, ring of 4: one round, fp32, 100 MiB 19 and 21, 400 MiB 76 and 78; plain gossip, fp32, 100 MiB 39
// and 38, 300 MiB 116 and 121, bf16 100 MiB 52 and 55; the D-PSGD step, fp32, 140 MiB 41 and 43, 800 MiB 250 and 238, bf16 204
// and 211; ring of 8, one round, bf16, 300 MiB 80 and 65.
enum Form : int { kGossipForm, kAtcForm, kAlg2Form, kDpsgdForm, kRoundForm };
inline uint64_t register_line(const Shape &s, int per_element, Form form) {
  const int64_t mib = footprint(s, per_element) >> 20;
  const bool few = s.n <= 8;
  if (s.n <= 4) {
    if (form == kRoundForm && mib >= 96) return 1;
    if (form == kGossipForm && mib >= (s.bf16 ? 96 : 128)) return 1;
    if (form == kDpsgdForm && mib >= 128 && (s.bf16 || mib < 200)) return 1;
  }
  if (!s.bf16) return 128;
  switch (form) {
    case kAtcForm: return few || s.n >= 48 || mib < 400 ? 64 : 128;
    case kRoundForm: return mib >= 96 && (few || mib < 200) ? 64 : 128;
    case kGossipForm: return mib >= 128 && few ? 64 : 128;
    default: return mib >= 128 && (few || mib < 280) ? 64 : 128;
  }
}

template <int N>
struct Ring {
  static constexpr int n = N, deg = 2;
  __host__ __device__ static constexpr int nb(int i, int k) { return k == 0 ? (i + N - 1) % N : (i + 1) % N; }
};

template <int R, int C>
struct Torus {
  static constexpr int n = R * C, deg = 4;
  __host__ __device__ static constexpr int nb(int i, int k) {
    const int r = i / C, c = i % C;
    return k == 0 ? ((r + R - 1) % R) * C + c
         : k == 1 ? ((r + 1) % R) * C + c
         : k == 2 ? r * C + (c + C - 1) % C
                  : r * C + (c + 1) % C;
  }
};

// The patterns the register-resident kernels are compiled for.  Calls f with a value of the pattern type that
// matches W (Ring<N> or Torus<R, C>) and returns its result; -1 if W is none of them.
template <class F>
int with_pattern(const HostW &W, F &&f) {
  if (W.structure == kRing) {
    switch (W.n) {
      case 4: return f(Ring<4>{});
      case 8: return f(Ring<8>{});
      case 12: return f(Ring<12>{});
      case 16: return f(Ring<16>{});
      case 24: return f(Ring<24>{});
      case 32: return f(Ring<32>{});
      case 48: return f(Ring<48>{});
      case 64: return f(Ring<64>{});
    }
  } else if (W.structure == kTorus) {
    if (W.trows == 8 && W.tcols == 8) return f(Torus<8, 8>{});
    if (W.trows == 4 && W.tcols == 4) return f(Torus<4, 4>{});
    if (W.trows == 4 && W.tcols == 8) return f(Torus<4, 8>{});
  }
  return -1;
}

// One round of Algorithm 3 in velocity form.  With v_r = z_r - z_{r-1} (v_0 = 0, since z_{-1} = z_0),
//   z_{r+1} = (1+eta) W^T z_r - eta z_{r-1}
// is the same as
//   v_{r+1,i} = b * sum_{j in nb(i)} (z_j - z_i) + eta * v_{r,i},   z_{r+1} = z_r + v_{r+1},   b = (1+eta)*w_nb
// (W_ii = 1 - deg*w_nb written out).  Two things make this the form to compute in fp32:
//  - a column whose workers all hold one value is a fixed point exactly, whatever the rounding of b and eta,
//    so the worker mean, which gradient tracking relies on, does not drift with the number of rounds;
//  - the only rounding at the magnitude of z is the final add; the recursion amplifies every rounding by up
//    to (1+(1+sqrt(eta))k) eta^(k/2) over the following k rounds, so fewer and smaller roundings matter
//    once eta is close to 1 (measured on 62 rounds at eta = 0.94: 2e-6 absolute against 1.3e-4 for
//    (1+eta)*(W_ii z_i + w_nb*sum) - eta*z_prev with separately rounded coefficients).
// Same operation count as that form (with the velocity kept divided by b, see ag_rounds).
struct Coef {
  float b, eta;
};

// sum of the neighbours' values, added pairwise so that deg equal values sum exactly
template <class T>
__device__ __forceinline__ float nb_sum(const float (&z)[T::n], int i) {
  static_assert(T::deg == 2 || T::deg == 4, "pairwise sum written for 2 or 4 neighbours");
  if constexpr (T::deg == 2) return z[T::nb(i, 0)] + z[T::nb(i, 1)];
  else return (z[T::nb(i, 0)] + z[T::nb(i, 1)]) + (z[T::nb(i, 2)] + z[T::nb(i, 3)]);
}

// sum_{j in nb(i)} (z_j - z_i)
template <class T>
__device__ __forceinline__ float lap(const float (&z)[T::n], int i) {
  return fmaf(-float(T::deg), z[i], nb_sum<T>(z, i));
}

// u <- eta * u + t as one three-operand instruction writing u's own register.  Left to the compiler, the
// loop-carried u becomes a two-operand v_fmac into t's register and a copy back: one instruction more per output
// and round, a seventh of the round loop.  The vector ALUs of these kernels are busy about two thirds of the time
// (counters), so the copy is not free everywhere, though on the machines where HBM sets the pace (3.9 ms for the
// gradient-fused step on the 8x8 torus at d = 11.2 M) taking it out measured no change.
__device__ __forceinline__ void momentum(float &u, float eta, float t) {
  asm("v_fma_f32 %0, %1, %0, %2" : "+v"(u) : "s"(eta), "v"(t));
}

// K >= 1 rounds starting from z_{-1} = z_0 = z.  Result in z; u is scratch: the velocity divided by b,
//   u_{r+1} = sum_nb (z_j - z_i) + eta * u_r,   z_{r+1} = z_r + b * u_{r+1},
// which is the recursion above with v = b*u and costs one multiplication less per output and round.
template <class T>
__device__ __forceinline__ void ag_rounds(float (&z)[T::n], float (&u)[T::n], const Coef &c, int K) {
#pragma unroll
  for (int i = 0; i < T::n; ++i) u[i] = lap<T>(z, i);
#pragma unroll
  for (int i = 0; i < T::n; ++i) z[i] = fmaf(c.b, u[i], z[i]);
  for (int r = 1; r < K; ++r) {
#pragma unroll
    for (int i = 0; i < T::n; ++i) momentum(u[i], c.eta, lap<T>(z, i));
#pragma unroll
    for (int i = 0; i < T::n; ++i) z[i] = fmaf(c.b, u[i], z[i]);
  }
}

// Register budget: the live state is 2 (gossip only) or 3 (phase) arrays of n
// floats per lane, plus the loads in flight.  The kernel asks for the matching
// waves-per-SIMD so the register allocator works against the real budget.
constexpr int waves_per_simd(int n, int mode) {
  const int need = n * (mode == 0 || mode == 3 ? 2 : 3) + 40;
  const int w = 512 / need;
  return w < 1 ? 1 : w > 8 ? 8 : w;
}

// Rows whose loads are in flight ahead of the row being consumed.  The loads
// of a tile are issued in row order through a software pipeline of this depth
// (the scheduling barriers pin that order); left alone, the compiler hoists all
// 4n loads of the tile to the top and spills.
// Measured on the 8x8 torus at d = 11.2 M: 4 to 15 rows ahead all give the same kernel time, 2 is 6 % slower.
constexpr int kRowsAhead = 12;

inline Coef make_coef(const HostW &W, float eta) {
  Coef c;
  c.b = float((1.0 + double(eta)) * W.w_nb);
  c.eta = eta;
  return c;
}

}  // namespace fused
}  // namespace detag
