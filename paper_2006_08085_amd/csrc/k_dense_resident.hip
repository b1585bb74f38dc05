// The dense phase of k_dense.hip with the rows of P resident in registers: bf16 state, and fp32 state of up to 128 workers.
//
// The general kernel fetches the rows of P with every tile, through the same in-order load counter as the state, so neither
// is hidden.  Here a block of eight wavefronts stays on its compute unit: each wavefront holds its 32 rows of P (two bf16
// terms, 8 KS registers a lane) for the whole call and walks tiles of 1024 / KS columns, so that a block always has 16 units
// of (16 workers x 64 columns) to stage, two to a wavefront.  The loads of the next units are in flight under the products of
// the present ones.
//
// Lane (m, g) of a unit loads columns 2m, 2m+1 of rows 8g..8g+7, which is what it holds of the B operand of two column tiles
// (even columns, odd columns).  So the terms go to LDS in fragment order, 16 bytes a lane (conflicts are a tenth of the
// LDS cycles), and an accumulator pair is one 32-bit word of two columns at the store: no transposition, one instruction moves
// 128 bytes of each of two rows.  Same products and order as the general kernel: the same values bit for bit where all are
// finite.  (State that is multiplied as it is stored is one term here, two there, the second of which is zero, or NaN beside
// an infinity.)
//
// Measured (K = 16, three states in turn, general kernel and this one): 256 workers, d = 1,000,000, pitch 1,000,064, ATC 1310
// and 911 us (4.5 TB/s), plain gossip 472 and 273; pitch 1,048,576, whose rows all start on the same
// memory channel, 1400 and 1063, 505 and 305; 128 workers, d = 2,000,000 1510 and 787 (5.2 TB/s: memory), 486 and 209; 64
// workers, d = 1,000,000 380 and 194, 102 and 50; 256 workers, d = 1,000 37 and 16, 15 and 7.5.  At 256 workers the matrix
// cores are busy 42 % of the time, the vector ALUs, with the staging, 19 %, and both wait at two barriers a tile; a deeper
// prefetch (one more quarter of the gradient rows) spills and loses, wavefront priorities change nothing.
#include "detag_internal.h"
#include "dev_common.hpp"
#include "fused_common.hpp"
#include "fused_generic_common.hpp"

namespace detag {
namespace {

constexpr int kThreads = 512, kWaves = 8, kUnits = 16;
constexpr int kMTiles = 8, kKSteps = 16;  // of the fragment order of P

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32_any __attribute__((aligned(2)));                        // two bf16 columns wherever they start
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));     // two fp32 columns

template <Access A>
__device__ __forceinline__ uint32_t load_pair(const char *base, uint32_t off) {
  const auto *p = reinterpret_cast<const u32_any *>(base + off);
  return A == kStream ? __builtin_nontemporal_load(p) : *p;
}
template <Access A>
__device__ __forceinline__ f32x2 load_two(const char *base, uint32_t off) {
  const auto *p = reinterpret_cast<const f32x2_any *>(base + off);
  return A == kStream ? __builtin_nontemporal_load(p) : *p;
}
template <Access A>
__device__ __forceinline__ float load_one(const char *base, uint32_t off) {
  const auto *p = reinterpret_cast<const float *>(base + off);
  return A == kStream ? __builtin_nontemporal_load(p) : *p;
}
template <Access A>
__device__ __forceinline__ void store_one(char *base, uint32_t off, float v) {
  auto *p = reinterpret_cast<float *>(base + off);
  if constexpr (A == kStream) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <Access A>
__device__ __forceinline__ void store_pair(char *base, uint32_t off, uint32_t v) {
  auto *p = reinterpret_cast<u32_any *>(base + off);
  if constexpr (A == kStream) __builtin_nontemporal_store(v, p);
  else *p = v;
}

__device__ __forceinline__ float low(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float high(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack(float a, float b) {  // both rounded to nearest even, a in the lower half
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The columns of a unit or of a wavefront's output, 64 from `col` on, `valid` of them (<= 0: none) inside the matrix.  A lane
// works on two adjacent columns from `at` on (relative to col); all of them are inside the matrix, so the last lanes of a
// ragged tile take columns twice and store nothing, or the second of theirs only.
struct Cols {
  int64_t col;
  int valid;
  uint32_t at;
  __device__ __forceinline__ Cols(int64_t c, int64_t d, int m) {
    const int v = int(d - c < 64 ? d - c : 64);
    const int c0 = 2 * m;
    valid = v;
    col = v == 1 ? c - 1 : c;  // a lone column: with the one before it, which is another tile's (d >= 64)
    at = v == 1 ? 0 : c0 + 1 < v ? c0 : c0 < v ? c0 - 1 : 0;
  }
  __device__ __forceinline__ bool both(int m) const { return 2 * m + 1 < valid; }
  __device__ __forceinline__ bool last(int m) const { return 2 * m + 1 == valid; }
};

// Rows of two columns a lane, `lane_rows` and up from wavefront-uniform row0 on, of `span` that the wavefront walks.  Rows past
// the last one repeat it: P is zero there, and what zero does not cancel (an infinity, a NaN) spoils its whole column anyway.
struct Rows {
  int64_t first;   // wavefront-uniform row the offsets count from
  bool full;       // wavefront-uniform: all `span` rows exist
  uint32_t start, step, lim;
  __device__ __forceinline__ Rows(int row0, int lane_rows, int span, int n, uint32_t pitch, uint32_t at, uint32_t size) {
    first = row0 < n ? row0 : n - 1;
    step = pitch * size;
    const int left = n - 1 - int(first);
    full = left >= span - 1 && row0 < n;
    lim = uint32_t(left < span - 1 ? left : span - 1) * step + at * size;
    start = uint32_t(lane_rows) * step + at * size;
  }
  // f(e, base of the row or of the first one, offset from there)
  template <int E0, int E1, class F>
  __device__ __forceinline__ void each(F &&f) const {
    if (full) {
#pragma unroll
      for (int e = 0; e < E1 - E0; ++e) f(e, uint64_t(E0 + e) * step, start);
    } else {
#pragma unroll
      for (int e = 0; e < E1 - E0; ++e) f(e, uint64_t(0), at(E0 + e));
    }
  }
  __device__ __forceinline__ uint32_t at(int e) const {
    const uint32_t o = start + uint32_t(e) * step;
    return o < lim ? o : lim;
  }
};

// The pitch, hidden from the optimiser: what follows from it is computed where it is used, with scalar instructions, instead of
// being kept for all rows across the walk over tiles.
__device__ __forceinline__ int64_t fresh(int64_t ld) {
  asm volatile("" : "+s"(ld));
  return ld;
}

// Two bf16 terms (both rounded to nearest) of 4 rows of a column: 8 bytes each.
__device__ __forceinline__ void split4(f32x4 v, uint2 &t0, uint2 &t1) {
  t0.x = pack(v[0], v[1]), t0.y = pack(v[2], v[3]);
  t1.x = pack(v[0] - low(t0.x), v[1] - high(t0.x)), t1.y = pack(v[2] - low(t0.y), v[3] - high(t0.y));
}

// The tiles of a block: every hop-th from `tile` to `last`.
template <Access A>
__device__ __forceinline__ void block_tiles(int tiles, int &tile, int &last, int &hop) {
  if (A == kKeep && gridDim.x % 8 == 0) {    // tiles that share cache lines: a contiguous eighth to every XCD
    const int per = (tiles + 7) / 8, x = blockIdx.x % 8;
    tile = x * per + blockIdx.x / 8, hop = gridDim.x / 8;
    last = (x + 1) * per < tiles ? (x + 1) * per : tiles;
  } else {
    tile = blockIdx.x, hop = gridDim.x, last = tiles;
  }
}

// mode 0: X <- P X.  mode 1 (ATC): X <- P (X - alpha*Y), Y <- P (Y + Gn - Go).
// mode 2 (ALG2): X <- P (X - alpha*Y), Y <- P Y + Gn - Go.  n <= 16 KS, d >= 64.
template <int MODE, int KS, Access A>
__global__ __launch_bounds__(kThreads, 2) void dense_resident_kernel(bf16_t *X, bf16_t *Y, const float *__restrict__ Gn,
                                                                  const float *__restrict__ Go, int n, int64_t d, int64_t ld,
                                                                  const u16x8 *__restrict__ frag, float alpha, int tiles) {
  constexpr int CT = kUnits / KS;            // sub-tiles of 64 columns in a tile
  constexpr int MT = KS / 2;                 // 32-row tiles of P
  constexpr bool kTwo = MODE != 0;           // X - alpha*Y
  extern __shared__ uint4 staged[];          // [pass or turn][unit][column tile][term][lane]
  uint4 *const lds_u = staged, *const lds_v = staged + kUnits * 256;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int mt = w % MT, osub = w / MT;      // this wavefront's output: 32 rows, one sub-tile

  u16x8 P[2][KS];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) P[t][s] = frag[((t * kMTiles + mt) * kKSteps + s) * 64 + lane];

  int tile, last, hop;
  block_tiles<A>(tiles, tile, last, hop);
  if (tile >= last) return;

  u32x8 lx[2], ly[2];                        // units w and w + 8
  using std::integral_constant;
  constexpr integral_constant<int, 0> k0{};
  constexpr integral_constant<int, 1> k1{};
  auto unit_cols = [&](int t, int k) { return Cols(int64_t(t) * (64 * CT) + 64 * ((w + 8 * k) % CT), d, m); };
  auto unit_rows = [&](int k, uint32_t pitch, uint32_t at, uint32_t size) {
    return Rows(16 * ((w + 8 * k) / CT), 8 * g, 16, n, pitch, at, size);
  };
  auto request_unit = [&](int t, auto k) {
    const Cols c = unit_cols(t, k);
    asm volatile("" : "=v"(lx[k]), "=v"(ly[k]));  // whatever: the old values must not stay alive for the case without a unit
    if (t >= last || c.valid <= 0) return;   // wavefront-uniform
    const int64_t l = fresh(ld);
    const Rows r = unit_rows(k, uint32_t(l), c.at, 2);
    const char *x = reinterpret_cast<const char *>(X + r.first * l + c.col);
    const char *y = reinterpret_cast<const char *>(Y + r.first * l + c.col);
    r.template each<0, 8>([&](int e, uint64_t row, uint32_t off) {
      lx[k][e] = load_pair<A>(x + row, off);
      if constexpr (kTwo) ly[k][e] = load_pair<A>(y + row, off);
    });
  };
  auto request_state = [&](int t) { request_unit(t, k0), request_unit(t, k1); };
  // A quarter of a wavefront's gradient rows (half a unit), and the tracker's terms of it -> LDS.
  f32x8 g0[2], g1[2];
  auto request_track = [&](int t, auto part, f32x8 (&to)[2]) {
    constexpr int k = part / 2, h = part % 2;
    const Cols c = unit_cols(t, k);
    asm volatile("" : "=v"(to[0]), "=v"(to[1]));
    if (t >= last || c.valid <= 0) return;
    const int64_t l = fresh(ld);
    const Rows r = unit_rows(k, uint32_t(l), c.at, 4);
    const char *a = reinterpret_cast<const char *>(Gn + r.first * l + c.col);
    const char *b = reinterpret_cast<const char *>(Go + r.first * l + c.col);
    r.template each<4 * h, 4 * h + 4>([&](int e, uint64_t row, uint32_t off) {
      const f32x2 p = load_two<A>(a + row, off), q = load_two<A>(b + row, off);
      to[0][2 * e] = p[0], to[0][2 * e + 1] = p[1], to[1][2 * e] = q[0], to[1][2 * e + 1] = q[1];
    });
  };
  auto stage_track = [&](auto part, const f32x8 (&from)[2]) {
    constexpr int k = part / 2, h = part % 2;
    f32x4 even, odd;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      even[e] = low(ly[k][4 * h + e]) + from[0][2 * e] - from[1][2 * e];
      odd[e] = high(ly[k][4 * h + e]) + from[0][2 * e + 1] - from[1][2 * e + 1];
    }
    uint2 *at = reinterpret_cast<uint2 *>(lds_v + (w + 8 * k) * 256 + lane) + h;
    uint2 t0, t1;
    split4(even, t0, t1);
    at[0] = t0, at[128] = t1;
    split4(odd, t0, t1);
    at[256] = t0, at[384] = t1;
    __builtin_amdgcn_sched_barrier(0);
  };
  // Waits for the state requested above.  Loads and stores are counted together and in order: without this, the first use
  // after the stores of a tile, whose number the compiler does not know, would wait for those as well.
  auto arrived = [&] {
    asm volatile("" : "+v"(lx[0]), "+v"(lx[1]));
    if constexpr (kTwo) asm volatile("" : "+v"(ly[0]), "+v"(ly[1]));
    if constexpr (MODE == 1) asm volatile("" : "+v"(g1[0]), "+v"(g1[1]));
  };
  // The state as it is stored is its own only term: half the room and two products of three.
  auto put_plain = [&](uint4 *lds, u32x8 v, int k) {
    uint4 *at = lds + (w + 8 * k) * 128 + lane;
    auto halves = [&](int e, uint32_t pick) { return __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], pick); };
    auto column = [&](uint32_t pick) { return make_uint4(halves(0, pick), halves(1, pick), halves(2, pick), halves(3, pick)); };
    at[0] = column(0x05040100u), at[64] = column(0x07060302u);
  };
  f32x16 acc[2];
  auto clear = [&] {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
  };
  // products with k-steps s0..s1-1, the smallest first; two: the staged input has two terms
  auto multiply = [&](const uint4 *lds, auto two, auto s0, auto s1) {
    constexpr int T = two ? 2 : 1;
#pragma unroll
    for (int s = s0; s < s1; ++s) {
      const uint4 *at = lds + (s * CT + osub) * (128 * T) + lane;
      u16x8 b[2][T];
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int t = 0; t < T; ++t) b[nt][t] = __builtin_bit_cast(u16x8, at[(nt * T + t) * 64]);
      constexpr int order[3][2] = {{0, 1}, {1, 0}, {0, 0}};
#pragma unroll
      for (int q = two ? 0 : 1; q < 3; ++q)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, P[order[q][0]][s]),
                                                            __builtin_bit_cast(bf16x8, b[nt][order[q][1]]), acc[nt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the wavefront's 32 rows of two columns a lane -> memory; fn(r) may change the pair of register r
  auto store_out = [&](bf16_t *out, int t, auto &&fn) {
    const Cols c(int64_t(t) * (64 * CT) + 64 * osub, d, m);
    if (c.valid <= 0 || 32 * mt >= n) return;
    const int64_t l = fresh(ld);
    const uint32_t step = uint32_t(l) * 2;
    char *base = reinterpret_cast<char *>(out + int64_t(32 * mt) * l + c.col);
    const uint32_t lane_off = 4 * g * step + 2 * c.at;
    if (c.valid == 64 && 32 * mt + 32 <= n) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float a = acc[0][r], b = acc[1][r];
        fn(r, a, b);
        store_pair<A>(base + int64_t(8 * (r / 4) + r % 4) * step, lane_off, pack(a, b));
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float a = acc[0][r], b = acc[1][r];
      fn(r, a, b);
      char *row = base + int64_t(8 * (r / 4) + r % 4) * step;
      if (32 * mt + 8 * (r / 4) + 4 * g + r % 4 < n) {
        const uint32_t v = pack(a, b);
        if (c.both(m)) store_pair<A>(row, lane_off, v);
        else if (c.last(m)) *reinterpret_cast<uint16_t *>(row + lane_off + 2) = uint16_t(v >> 16);
      }
    }
  };
  constexpr integral_constant<int, KS> kAll{};
  constexpr integral_constant<bool, true> kBoth{};
  [[maybe_unused]] int turn = 0;
  auto plain = [](int, float &, float &) {};

  request_state(tile);
  if constexpr (MODE == 1) request_track(tile, k0, g1);
  for (; tile < last; tile += hop) {
    const int next = tile + hop;
    if constexpr (MODE == 0) {
      // two buffers in turn: who is here has passed the barrier behind the last products with this one
      uint4 *const lds = staged + turn * kUnits * 128;
      turn ^= 1;
      put_plain(lds, lx[0], k0), put_plain(lds, lx[1], k1);
      request_state(next);
      __syncthreads();
      clear();
      multiply(lds, integral_constant<bool, false>{}, k0, kAll);
      arrived();
      store_out(X, tile, plain);
    } else {
      auto stage_model = [&](auto k) {
        f32x8 even, odd;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          even[e] = fmaf(-alpha, low(ly[k][e]), low(lx[k][e]));
          odd[e] = fmaf(-alpha, high(ly[k][e]), high(lx[k][e]));
        }
        uint4 *at = lds_u + (w + 8 * k) * 256 + lane;
        auto column = [&](int o, f32x8 v) {
          uint2 a0, a1, b0, b1;
          split4(v.lo, a0, a1), split4(v.hi, b0, b1);
          at[o] = make_uint4(a0.x, a0.y, b0.x, b0.y), at[o + 64] = make_uint4(a1.x, a1.y, b1.x, b1.y);
        };
        column(0, even), column(128, odd);
      };
      stage_model(k0), stage_model(k1);
      if constexpr (MODE == 1) {
        __syncthreads();                     // the terms of X - alpha*Y are in place, those of the last tracker are done with
        stage_track(k0, g1);
        request_track(tile, k1, g0);
        request_track(tile, integral_constant<int, 2>{}, g1);
        __builtin_amdgcn_sched_barrier(0);
        clear();
        multiply(lds_u, kBoth, k0, integral_constant<int, KS / 2>{});
        stage_track(k1, g0);
        request_track(tile, integral_constant<int, 3>{}, g0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(lds_u, kBoth, integral_constant<int, KS / 2>{}, integral_constant<int, KS * 3 / 4>{});
        stage_track(integral_constant<int, 2>{}, g1);
        multiply(lds_u, kBoth, integral_constant<int, KS * 3 / 4>{}, kAll);
        stage_track(integral_constant<int, 3>{}, g0);
      } else {
        __syncthreads();
        put_plain(lds_v, ly[0], k0), put_plain(lds_v, ly[1], k1);
        clear();
        multiply(lds_u, kBoth, k0, kAll);
      }
      request_state(next);
      if constexpr (MODE == 1) request_track(next, k0, g1);
      __builtin_amdgcn_sched_barrier(0);
      store_out(X, tile, plain);
      __syncthreads();                       // the terms of the tracker are in place, those of the model are done with
      clear();
      multiply(lds_v, integral_constant<bool, MODE == 1>{}, k0, kAll);
      arrived();
      if constexpr (MODE == 1) {
        store_out(Y, tile, plain);
      } else {
        const Cols c(int64_t(tile) * (64 * CT) + 64 * osub, d, m);
        if (c.valid > 0 && 32 * mt < n) {
          // register r: row 32 mt + 8 (r / 4) + 4 g + r % 4; four rows ahead of the stores
          const int64_t l = fresh(ld);
          const Rows q(32 * mt, 4 * g, 32, n, uint32_t(l), c.at, 4);
          const char *a = reinterpret_cast<const char *>(Gn + q.first * l + c.col);
          const char *b = reinterpret_cast<const char *>(Go + q.first * l + c.col);
          f32x2 wn[16], wo[16];
          auto ahead = [&](int r) {
            const int e = 8 * (r / 4) + r % 4;
            wn[r] = load_two<A>(a, q.at(e)), wo[r] = load_two<A>(b, q.at(e));
          };
#pragma unroll
          for (int r = 0; r < 4; ++r) ahead(r);
          store_out(Y, tile, [&](int r, float &even, float &odd) {
            if (r + 4 < 16) ahead(r + 4);
            even = even + wn[r][0] - wo[r][0], odd = odd + wn[r][1] - wo[r][1];
            __builtin_amdgcn_sched_barrier(0);
          });
        }
      }
    }
  }
}

// The same for fp32 state and up to 128 workers: three terms and six products, as the general kernel cuts and orders them.
// Three terms of P for 256 workers would fill the register file.  A block stages 8 units, one to a wavefront, and a wavefront
// multiplies for 32 rows of one column tile (the first or the second 32 columns of a sub-tile): two passes of 48 KiB.
// Measured (K = 16, three states in turn, general kernel and this one): 128 workers, d = 409,600, ATC 537 and 269 us (4.7
// TB/s), pitch 409,601 636 and 321, plain gossip 128 and 101; 64 workers, d = 819,200 342 and 249, Algorithm 2's phase 516 and
// 266; 20 workers, d = 2,621,440 384 and 258; 100 workers, d = 1,000 25 and 10.
__device__ __forceinline__ void split4(f32x4 v, uint2 (&t)[3]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    auto upper = [&](int e) { return __builtin_amdgcn_perm(__float_as_uint(v[e + 1]), __float_as_uint(v[e]), 0x07060302u); };
    t[p] = make_uint2(upper(0), upper(2));
    if (p < 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] -= __uint_as_float(__float_as_uint(v[e]) & 0xffff0000u);
    }
  }
}

template <int MODE, int KS, Access A>
__global__ __launch_bounds__(kThreads, 2) void dense_resident_f32_kernel(float *X, float *Y, const float *__restrict__ Gn,
                                                                      const float *__restrict__ Go, int n, int64_t d,
                                                                      int64_t ld, const u16x8 *__restrict__ frag, float alpha,
                                                                      int tiles) {
  constexpr int CT = kWaves / KS;            // sub-tiles of 64 columns in a tile
  constexpr int MT = KS / 2;                 // 32-row tiles of P
  constexpr bool kTwo = MODE != 0;
  constexpr int kUnit = 2 * 3 * 64;          // 16-byte words of a unit: column tiles, terms, lanes
  extern __shared__ uint4 staged[];          // [pass or turn][unit][column tile][term][lane]
  uint4 *const lds_u = staged, *const lds_v = staged + kWaves * kUnit;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 31, g = lane >> 5;
  const int mt = w % MT, osub = w / MT % CT, ont = w / (MT * CT);  // this wavefront's output
  const int step_of = w / CT, sub_of = w % CT;                      // the unit it stages

  u16x8 P[3][KS];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) P[t][s] = frag[((t * kMTiles + mt) * kKSteps + s) * 64 + lane];

  int tile, last, hop;
  block_tiles<A>(tiles, tile, last, hop);
  if (tile >= last) return;

  // The lane's column of a sub-tile's column tile, repeating the last one (relative to the sub-tile).
  auto column = [&](int valid, int nt) { return uint32_t(32 * nt + m < valid ? 32 * nt + m : valid - 1); };
  auto valid_of = [&](int t, int sub) {
    const int64_t left = d - (int64_t(t) * (64 * CT) + 64 * sub);
    return int(left < 64 ? left : 64);
  };
  f32x8 lx[2], ly[2];                        // column tile, row
  auto request = [&](const float *Z, int t, auto e0, auto e1, auto &&put) {
    const int valid = valid_of(t, sub_of);
    const int64_t l = fresh(ld);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const Rows r(16 * step_of, 8 * g, 16, n, uint32_t(l), column(valid, nt), 4);
      const char *z = reinterpret_cast<const char *>(Z + r.first * l + int64_t(t) * (64 * CT) + 64 * sub_of);
      r.template each<e0, e1>([&](int e, uint64_t row, uint32_t off) { put(nt, e, load_one<A>(z + row, off)); });
    }
  };
  using std::integral_constant;
  constexpr integral_constant<int, 0> k0{};
  constexpr integral_constant<int, 4> k4{};
  constexpr integral_constant<int, 8> k8{};
  auto exists = [&](int t) { return t < last && valid_of(t, sub_of) > 0; };  // wavefront-uniform
  auto request_state = [&](int t) {
    asm volatile("" : "=v"(lx[0]), "=v"(lx[1]), "=v"(ly[0]), "=v"(ly[1]));
    if (!exists(t)) return;
    request(X, t, k0, k8, [&](int nt, int e, float v) { lx[nt][e] = v; });
    if constexpr (kTwo) request(Y, t, k0, k8, [&](int nt, int e, float v) { ly[nt][e] = v; });
  };
  f32x8 g0[2], g1[2];                        // half the rows: new and old gradient, [column tile * 4 + row]
  auto request_track = [&](int t, auto half, f32x8 (&to)[2]) {
    asm volatile("" : "=v"(to[0]), "=v"(to[1]));
    if (!exists(t)) return;
    constexpr integral_constant<int, 4 * half> from{};
    constexpr integral_constant<int, 4 * half + 4> end{};
    request(Gn, t, from, end, [&](int nt, int e, float v) { to[0][4 * nt + e] = v; });
    request(Go, t, from, end, [&](int nt, int e, float v) { to[1][4 * nt + e] = v; });
  };
  auto put_half = [&](uint4 *lds, int nt, int half, f32x4 v) {
    uint2 t[3];
    split4(v, t);
    uint2 *at = reinterpret_cast<uint2 *>(lds + w * kUnit + nt * 192 + lane) + half;
#pragma unroll
    for (int p = 0; p < 3; ++p) at[p * 128] = t[p];
  };
  auto put = [&](uint4 *lds, int nt, f32x8 v) {
    uint2 a[3], b[3];
    split4(v.lo, a), split4(v.hi, b);
    uint4 *at = lds + w * kUnit + nt * 192 + lane;
#pragma unroll
    for (int p = 0; p < 3; ++p) at[p * 64] = make_uint4(a[p].x, a[p].y, b[p].x, b[p].y);
  };
  auto stage_track = [&](auto half, const f32x8 (&from)[2]) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = ly[nt][4 * half + e] + from[0][4 * nt + e] - from[1][4 * nt + e];
      put_half(lds_v, nt, half, v);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto arrived = [&] {
    asm volatile("" : "+v"(lx[0]), "+v"(lx[1]));
    if constexpr (kTwo) asm volatile("" : "+v"(ly[0]), "+v"(ly[1]));
    if constexpr (MODE == 1) asm volatile("" : "+v"(g0[0]), "+v"(g0[1]));
  };
  f32x16 acc;
  auto clear = [&] {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  };
  auto multiply = [&](const uint4 *lds, auto s0, auto s1) {
#pragma unroll
    for (int s = s0; s < s1; ++s) {
      const uint4 *at = lds + (s * CT + osub) * kUnit + ont * 192 + lane;
      u16x8 b[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) b[t] = __builtin_bit_cast(u16x8, at[t * 64]);
      constexpr int order[6][2] = {{0, 2}, {1, 1}, {2, 0}, {0, 1}, {1, 0}, {0, 0}};
#pragma unroll
      for (int q = 0; q < 6; ++q)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, P[order[q][0]][s]),
                                                      __builtin_bit_cast(bf16x8, b[order[q][1]]), acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // fn(r, value) may change the value of register r on its way
  auto store_out = [&](float *out, int t, auto &&fn) {
    const int valid = valid_of(t, osub);
    if (valid <= 0 || 32 * mt >= n) return;
    const int64_t l = fresh(ld);
    const uint32_t step = uint32_t(l) * 4;
    char *base = reinterpret_cast<char *>(out + int64_t(32 * mt) * l + int64_t(t) * (64 * CT) + 64 * osub);
    const uint32_t lane_off = 4 * g * step + 4 * (32 * ont + m);
    const bool whole = valid == 64 && 32 * mt + 32 <= n;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = fn(r, acc[r]);
      char *row = base + int64_t(8 * (r / 4) + r % 4) * step;
      if (whole || (32 * ont + m < valid && 32 * mt + 8 * (r / 4) + 4 * g + r % 4 < n)) store_one<A>(row, lane_off, v);
    }
  };
  auto plain = [](int, float v) { return v; };
  constexpr integral_constant<int, KS / 2> kHalf{};
  constexpr integral_constant<int, KS> kAll{};
  [[maybe_unused]] int turn = 0;

  request_state(tile);
  if constexpr (MODE == 1) request_track(tile, k0, g0);
  for (; tile < last; tile += hop) {
    const int next = tile + hop;
    if constexpr (MODE == 0) {
      uint4 *const lds = staged + turn * kWaves * kUnit;
      turn ^= 1;
      put(lds, 0, lx[0]), put(lds, 1, lx[1]);
      request_state(next);
      __syncthreads();
      clear();
      multiply(lds, k0, kAll);
      arrived();
      store_out(X, tile, plain);
    } else {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        f32x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = fmaf(-alpha, ly[nt][e], lx[nt][e]);
        put(lds_u, nt, v);
      }
      __syncthreads();                       // the terms of X - alpha*Y are in place, those of the last tracker are done with
      if constexpr (MODE == 1) {
        stage_track(k0, g0);
        request_track(tile, integral_constant<int, 1>{}, g1);
        __builtin_amdgcn_sched_barrier(0);
        clear();
        multiply(lds_u, k0, kAll);
        stage_track(integral_constant<int, 1>{}, g1);
      } else {
        put(lds_v, 0, ly[0]), put(lds_v, 1, ly[1]);
        clear();
        multiply(lds_u, k0, kAll);
      }
      request_state(next);
      if constexpr (MODE == 1) request_track(next, k0, g0);
      __builtin_amdgcn_sched_barrier(0);
      store_out(X, tile, plain);
      __syncthreads();                       // the terms of the tracker are in place, those of the model are done with
      clear();
      multiply(lds_v, k0, kAll);
      arrived();
      if constexpr (MODE == 1) {
        store_out(Y, tile, plain);
      } else {
        const int valid = valid_of(tile, osub);
        if (valid > 0 && 32 * mt < n) {
          const int64_t l = fresh(ld);
          const Rows q(32 * mt, 4 * g, 32, n, uint32_t(l), column(valid, ont), 4);
          const int64_t off = q.first * l + int64_t(tile) * (64 * CT) + 64 * osub;
          const char *a = reinterpret_cast<const char *>(Gn + off), *b = reinterpret_cast<const char *>(Go + off);
          f32x16 wn, wo;
          auto ahead = [&](int r) {
            const int e = 8 * (r / 4) + r % 4;
            wn[r] = load_one<A>(a, q.at(e)), wo[r] = load_one<A>(b, q.at(e));
          };
#pragma unroll
          for (int r = 0; r < 8; ++r) ahead(r);
          store_out(Y, tile, [&](int r, float v) {
            if (r + 8 < 16) ahead(r + 8);
            const float o = v + wn[r] - wo[r];
            __builtin_amdgcn_sched_barrier(0);
            return o;
          });
        }
      }
    }
  }
}

template <int KS, Access A>
int launch_ks(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, float alpha, const uint16_t *frag,
              hipStream_t st) {
  constexpr int cols = 64 * (kUnits / KS);
  const int tiles = ceil_div_i64(s.d, cols);
  const int grid = tiles < 256 ? tiles : 256;  // one block to a compute unit
  const size_t lds = size_t(mode == 0 ? 256 : mode == 1 ? 512 : 384) * kUnits * sizeof(uint4);
  auto go = [&](auto *kernel) -> int {
    if (int rc = lds_tile::allow_lds(reinterpret_cast<const void *>(kernel), lds)) return rc;
    kernel<<<grid, kThreads, lds, st>>>(static_cast<bf16_t *>(X), static_cast<bf16_t *>(Y), Gn, Go, s.n, s.d, s.ld,
                                        reinterpret_cast<const u16x8 *>(frag), alpha, tiles);
    return hip_rc(hipGetLastError());
  };
  switch (mode) {
    case 0: return go(&dense_resident_kernel<0, KS, A>);
    case 1: return go(&dense_resident_kernel<1, KS, A>);
    default: return go(&dense_resident_kernel<2, KS, A>);
  }
}

template <int KS, Access A>
int launch_f32(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, float alpha, const uint16_t *frag,
               hipStream_t st) {
  const int tiles = ceil_div_i64(s.d, 64 * (kWaves / KS));
  const int grid = tiles < 256 ? tiles : 256;
  const size_t lds = 2 * size_t(kWaves) * 2 * 3 * 64 * sizeof(uint4);
  auto go = [&](auto *kernel) -> int {
    if (int rc = lds_tile::allow_lds(reinterpret_cast<const void *>(kernel), lds)) return rc;
    kernel<<<grid, kThreads, lds, st>>>(static_cast<float *>(X), static_cast<float *>(Y), Gn, Go, s.n, s.d, s.ld,
                                        reinterpret_cast<const u16x8 *>(frag), alpha, tiles);
    return hip_rc(hipGetLastError());
  };
  switch (mode) {
    case 0: return go(&dense_resident_f32_kernel<0, KS, A>);
    case 1: return go(&dense_resident_f32_kernel<1, KS, A>);
    default: return go(&dense_resident_f32_kernel<2, KS, A>);
  }
}

template <Access A>
int launch_access(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, float alpha,
                  const uint16_t *frag, hipStream_t st) {
  if (!s.bf16) {
    if (s.n <= 32) return launch_f32<2, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
    if (s.n <= 64) return launch_f32<4, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
    return launch_f32<8, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
  }
  if (s.n <= 32) return launch_ks<2, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
  if (s.n <= 64) return launch_ks<4, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
  if (s.n <= 128) return launch_ks<8, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
  return launch_ks<16, A>(s, mode, X, Y, Gn, Go, alpha, frag, st);
}

}  // namespace

// What this kernel takes: lanes count their offsets within 32 rows of fp32 in 32 bits, a lone last column is loaded with the one
// before it, and the P of a call is read by every block before its first tile, which the smallest calls of few workers notice
// (general kernel and this one, replayed, K = 4: ATC phase, 12 workers, fp32, d = 1,000 5.6 and 6.2 us, 16,000 5.9 and 6.5,
// 26,000 6.4 and 6.5, 16 workers 5.8 and 6.3, 6.1 and 6.6, 17 level; bf16, d = 1,000 6.8 and 7.6, 16,000 6.9 and 7.6, 50,000
// 10.3 and 7.8; plain gossip of 32 workers, bf16, d = 1,000 4.9 and 5.2, 16,000 5.0 and 5.3, 50,000 6.4 and 5.2, fp32 4.5 and
// 4.9, 4.6 and 4.9, 6.6 and 5.4; Algorithm 2's phase of 5, bf16, d = 8,000 5.7 and 6.3, of 7 6.1 and 6.4, of 8 level, fp32 within
// 4 % both ways).
bool dense_resident_serves(const Shape &s, int mode) {
  if (!s.bf16 && s.n > 128) return false;
  if (s.d < 64 || s.ld > (int64_t(1) << 25)) return false;
  const int few = mode == 0 ? 32 : mode == 1 ? 16 : s.bf16 ? 7 : 0;
  return s.n > few || s.d >= (mode == 0 || (mode == 1 && s.bf16) ? 32768 : 20480);
}

int launch_dense_resident(const Shape &s, int mode, void *X, void *Y, const float *Gn, const float *Go, float alpha,
                          const uint16_t *frag, void *stream) {
  auto st = static_cast<hipStream_t>(stream);
  // Tiles that share cache lines go to one XCD and leave their accesses to the caches (streamed and kept, ATC: 256 x 200,001
  // 316 and 213 us, 64 x 546,113 164 and 128, 20 x 1,747,585 166 and 143), and so do calls that the memory-side cache serves
  // (256 workers, 60 MiB 31.0 and 27.7, 100 MiB 44.2 and 43.3, 130 MiB 47.0 and 47.0, 200 MiB 75.1 and 79.4; 64 workers 80 MiB
  // 24.3 and 22.3, 200 MiB 57.3 and 66.2; fp32, 128 workers 100 MiB 43.2 and 42.0, 140 MiB 54.9 and 58.0; Algorithm 2's phase
  // the same; plain gossip of 256 workers, 33 MiB 25.5 and 24.3, 95 MiB of 64 and 100 workers 49.6 and 53.1, 95.5 and 97.5, fp32
  // 50 MiB 24.7 and 21.6, 200 MiB 82.4 and 91.4).
  const int64_t bytes = fused::footprint(s, (mode == 0 ? 1 : 2) * (s.bf16 ? 2 : 4) + (mode == 0 ? 0 : 8));
  const bool keep = fused::shares_lines(s, {X, Y, Gn, Go}) || bytes <= (int64_t(mode == 0 ? 64 : 104) << 20);
  return keep ? launch_access<kKeep>(s, mode, X, Y, Gn, Go, alpha, frag, st)
              : launch_access<kStream>(s, mode, X, Y, Gn, Go, alpha, frag, st);
}

}  // namespace detag
