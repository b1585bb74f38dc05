// Shared by the LDS-resident kernels: the K-round fused DeTAG phase for a sparse gossip matrix without compile-time
// structure (a random regular graph, a user's own network, rings and tori off the register family's list).
//
// A block owns `cols` (16 ... 256) adjacent columns and all n rows of them.  A lane owns FOUR ADJACENT columns of S rows:
// cols/4 lanes side by side cover a row, a wavefront 256/cols rows, and lane t of a block of T threads owns the rows at
// LDS offsets 16 t + 16 T s, s < S.  z_r and the velocity of its rows stay in registers; z_r of all rows also sits in
// LDS, where the neighbours of a row are read: one round = read the neighbours, barrier, write the new values back,
// barrier.  HBM sees the state once per phase (24 B per element with fp32 state, 16 B with bf16, whatever K is).
//
// Why four columns per lane: the rounds are bound by LDS traffic, (deg + 1) words per output, and gfx950's LDS
// delivers 240 B per clock and compute unit to 16-byte reads but 116 to 4-byte reads (measured; with the one write
// per four reads of a 4-regular graph 174 against 98).  A read also needs one address per four outputs instead of
// one per output.  With one column per lane (and one row per wavefront, so that row offsets were scalars) the step of
// the 256-worker workload took 3.14 ms; now 2.12 ms, of which the rounds (26.5 us for 64 Mi elements of X and Y) run
// at the rate the LDS and the vector ALUs, about equally busy, allow.
//
// S = 4 is the form for matrices that fill the chip.  S = 1 and 2 spread a small matrix over more wavefronts: its time
// is the length of the chain load - K rounds - store, so a lane does less, keeps its neighbour list in registers, and
// the rounds alternate between two tiles in LDS, which saves one of the two barriers.
//
// Forms of the neighbour table:
//   ByteRounds<DEG, S>  n <= 256, at most 8 neighbours, one weight for the whole matrix (any regular graph with uniform
//                    or Metropolis weights): a neighbour is one byte, the high byte of its row's LDS offset, so the table
//                    of a row is DEG/4 registers and an address is one byte permute.
//   HalfRounds<DEG>  the same with more than 256 workers and S = 4: two bytes per neighbour.
//   ListRounds<S>    any weights, at most 8 neighbours, S < 4: the row's (offset, weight) pairs in registers.
//   CsrRounds<S>     any weights and degrees, n <= 1024: the rows' lists sit in LDS next to the tile as pairs of (offset,
//                    weight), two per 16-byte read, which all lanes of a row read together.  The host orders the
//                    rows by degree, so that the rows a wavefront walks together have lists of about one length.
// All evaluate a round in velocity form, v = z_r - z_{r-1},
//   v_i <- (1+eta) * sum_j W_ji (z_j - z_i) + eta * v_i,   z_i <- z_i + v_i,
// in which equal values across the workers are a fixed point exactly whatever the rounding of the weights (the worker
// mean does not drift with K) and the only rounding at the magnitude of z is the last add.
//
// The ByteRounds kernels with S = 4 are kept within 64 VGPRs (three arrays of 16 values per lane in a phase), so that 32
// wavefronts share a compute unit: one block's loads and stores run under the other blocks' rounds.
//
// Paper: Algorithm 3 (accelerated gossip) and Algorithm 2 / the matrix form in
// the proof of Theorem 3 (phase update).
#pragma once

#include <type_traits>

#include "detag_internal.h"
#include "dev_common.hpp"
#include "fused_common.hpp"

namespace detag {
namespace lds_tile {

constexpr int kSlotsMax = 4;         // rows per lane (S above)
constexpr int kThreadsMax = 1024;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
// the same for rows that start anywhere (an odd pitch): one access all the same, memory needs no 16-byte alignment
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u2_any __attribute__((ext_vector_type(2), aligned(2)));  // four bf16 values

template <Access A>
__device__ __forceinline__ f4 load4(const float *p) {
  const f4_any *q = reinterpret_cast<const f4_any *>(p);
  return A == kStream ? __builtin_nontemporal_load(q) : *q;
}
template <Access A>
__device__ __forceinline__ u2 load4(const bf16_t *p) {
  const u2_any *q = reinterpret_cast<const u2_any *>(p);
  return A == kStream ? __builtin_nontemporal_load(q) : *q;
}
// What a load brought, as floats: next to the use, since whatever touches it waits for it.
__device__ __forceinline__ f4 floats(f4 v) { return v; }
__device__ __forceinline__ f4 floats(u2 t) {
  f4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(e & 1 ? t[e / 2] & 0xffff0000u : t[e / 2] << 16);
  return v;
}
template <class ST>
using Raw = std::conditional_t<std::is_same_v<ST, float>, f4, u2>;
template <Access A>
__device__ __forceinline__ void store4(float *p, f4 v) {
  f4_any *q = reinterpret_cast<f4_any *>(p);
  if constexpr (A != kKeep) __builtin_nontemporal_store(f4_any(v), q);
  else *q = v;
}
template <Access A>
__device__ __forceinline__ void store4(bf16_t *p, f4 v) {
  const u2 t = {bf16_bits_rne(v[0]) | uint32_t(bf16_bits_rne(v[1])) << 16, bf16_bits_rne(v[2]) | uint32_t(bf16_bits_rne(v[3])) << 16};
  u2_any *q = reinterpret_cast<u2_any *>(p);
  if constexpr (A != kKeep) __builtin_nontemporal_store(u2_any(t), q);
  else *q = t;
}

// The columns of a block: all exist; the rows end after four of them or more; after fewer than four.
enum Tile : int { kNarrow, kCut, kWhole };

// The four columns of a lane.  Columns are independent, so in a cut tile a lane whose columns do not all exist takes the
// row's last four instead (at = d - 4): those before its own are computed once more and not stored, a lane past the end
// stores none.  The accesses are those of a whole tile.  One by one, with a 64-bit address for each column, the cut tile
// was so much code that fetching it took longer than the rest of a small call (1000 workers on a ring, d = 300, K = 4
// 51 us, 23 us so; 256 workers, 4-regular, d = 3,915, K = 1 14.9 and 8.0 us).  A narrow tile is read one by one: its row's
// last four columns lie in lines of the tile before (d = 3,906 8.4 us, 10.9 us the other way).
struct Columns {
  int64_t at;  // the first of them
  int skip;    // how many of them belong to the lane before; 4 or more: none is the lane's
};

// How a block's columns lie.  CUT = false: cut tiles are treated like narrow ones.  IN_SGPR: one scalar register decides
// for all of a block's loads and stores, which saves the kernels that live within 64 vector registers a spill in their
// rounds; without it the compiler lays the whole tiles' code out as the straight path, which is 2 to 10 % of a phase where
// one block of 1024 threads has a compute unit to itself (1000 workers, d = 60,000, K = 1 387 and 404 us).
template <bool CUT, bool IN_SGPR>
__device__ __forceinline__ int tile_kind(int64_t first, int lpr_log2, int64_t d) {
  const int64_t left = d - first;
  const bool whole = left >= int64_t(4) << lpr_log2;
  if constexpr (!CUT) return whole ? kWhole : kNarrow;
  if constexpr (IN_SGPR) return __builtin_amdgcn_readfirstlane(whole ? kWhole : left >= 4 ? kCut : kNarrow);
  return whole ? kWhole : left >= 4 ? kCut : kNarrow;
}

template <int TILE, Access A, class ST>
__device__ __forceinline__ Raw<ST> load4(const ST *base, int64_t row_off, const Columns &c, int64_t d) {
  if constexpr (TILE != kNarrow) return load4<A>(base + (row_off + c.at));
  auto one = [&](int e) { return base[row_off + (c.at + e < d ? c.at + e : d - 1)]; };  // columns past the last repeat it
  if constexpr (std::is_same_v<ST, float>) return f4{one(0), one(1), one(2), one(3)};
  else return u2{one(0).bits | uint32_t(one(1).bits) << 16, one(2).bits | uint32_t(one(3).bits) << 16};
}
template <int TILE, Access A, class ST>
__device__ __forceinline__ void store4(ST *base, int64_t row_off, const Columns &c, int64_t d, f4 v) {
  if (TILE == kWhole || (TILE == kCut && c.skip == 0)) {
    store4<A>(base + (row_off + c.at), v);
  } else {
#pragma unroll
    for (int e = TILE == kCut; e < 4; ++e)
      if (e >= c.skip && (TILE == kCut || c.at + e < d)) base[row_off + c.at + e] = from_f32<ST>(v[e]);
  }
}

__device__ __forceinline__ f4 fma4(float a, f4 b, f4 c) {
  f4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = fmaf(a, b[e], c[e]);
  return r;
}

__device__ __forceinline__ void pin4(f4 &v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float t = v[e];
    pin_vgpr(t);
    v[e] = t;
  }
}

// The tile starts at LDS offset 0: the kernels have no other LDS (tests/test_kernel_metadata.py).  Addressed as numbers,
// an access costs no addition of a base that is zero.
typedef __attribute__((address_space(3))) f4 lds_f4;
__device__ __forceinline__ f4 lds_read(uint32_t off) { return *reinterpret_cast<const lds_f4 *>(off); }
__device__ __forceinline__ void lds_write(uint32_t off, f4 v) { *reinterpret_cast<lds_f4 *>(off) = v; }

// Where a lane sits: its column (in the block's tile) and its position among the rows of a slot.
struct Place {
  uint32_t tid, threads;
  int lpr_log2;  // lanes per row = cols / 4
  __device__ __forceinline__ uint32_t col() const { return (tid & ((1u << lpr_log2) - 1u)) * 4u; }
  __device__ __forceinline__ uint32_t pos(int s) const { return (tid + s * threads) >> lpr_log2; }
  __device__ __forceinline__ uint32_t own(int s) const { return (tid + s * threads) * 16u; }
  // What was derived from tid so far (row addresses, LDS offsets) is derived anew from here on instead of being kept.
  __device__ __forceinline__ void forget() { asm volatile("" : "+v"(tid)); }
};

// Blocks of S < 4 hold two tiles; the second one starts here (a compile-time distance, so that it costs no address).
constexpr uint32_t second_tile(int S) { return uint32_t(S) * kThreadsMax * 16u; }

// A small matrix is a chain of memory latencies: the table of its S < 4 rows per lane is requested ahead of the state
// (13 irregular workers, d = 7,692, K = 4 7.3 -> 6.7 us).  With S = 4 its registers are free for the first loads and it
// comes after them.
template <int S>
constexpr bool kFetchFirst = S < kSlotsMax;
// Rows requested ahead of the one in use, where a row is four or five arrays (PLENTY of two arrays or four; with the noise
// one less).  A lane's rows one after the other, each waiting for its own loads, were the memory phases of these kernels:
// half of the blocks of a compute unit are in their rounds, and the others did not keep the memory busy.  Within 64 registers
// one row fits ahead, none beside the noise, whose Philox state then spills (bf16 values unpacked next to their loads took
// two registers to one and spilled 22).  One by one and ahead: phase, 300 workers, 4-regular, d = 100,000, K = 8 fp32 253 ->
// 240 us, K = 2, bf16 140 -> 115; fused step, 100 irregular workers, d = 500,000, K = 8 460 -> 425, 30, d = 1,000,000, K = 3,
// bf16 158 -> 135, 64 workers, 4-regular, d = 1,000,000, K = 8 375 -> 368, 24 irregular workers, d = 3,000, K = 4 with its
// gradient 12.7 -> 10.9.  The fused step of few workers with one weight, fp32, K <= 4, whose call just outgrows the caches, pays
// for it (64 workers, 4 and 8 neighbours, 4.5 Mi elements, K = 1 and 2 4 to 8 %) and gains elsewhere.
constexpr int kInOneGo = -1;  // a row's loads and their use between the same two fences
template <class R, int PLENTY>
constexpr int kAhead = R::kSlots < kSlotsMax ? R::kSlots - 1 : PLENTY - (R::kWaves == 8);

template <int DEG, int S>
struct ByteRounds {
  static constexpr int kSlots = S, kWords = DEG <= 4 ? 1 : DEG / 4;
  static constexpr int kWaves = S == 4 ? 8 : 4;  // wavefronts per SIMD asked of the register allocator
  static constexpr int kParked = S == 4 ? 1 : 0;
  static constexpr bool kRowsInMemory = false;
  struct Args {
    const uint32_t *table;  // kWords words per row, 256 rows: one byte per neighbour, its row number
    float weight;
  };
  uint32_t w[S][kWords];
  uint32_t low;  // low byte of the lane's column offset
  float b;

  __device__ __forceinline__ void fetch(const Args &a, const Place &p) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int q = 0; q < kWords; ++q) w[s][q] = a.table[p.pos(s) * kWords + q];
  }
  __device__ __forceinline__ void init(const Args &a, const Place &p, float eta) {
    if constexpr (!kFetchFirst<S>) fetch(a, p);
    // row r starts at r * cols * 4 bytes and the columns add up to cols * 4 - 1: the neighbour's byte becomes bits 8..15
    // of the address of the lane's columns in that row (cols is 64, 128 or 256; n * cols <= 16384)
    const uint32_t byte_col = p.col() * 4u, scale = 1u << (p.lpr_log2 - 4);
    low = byte_col & 0xffu;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int q = 0; q < kWords; ++q) w[s][q] = w[s][q] * scale + (byte_col >> 8) * 0x01010101u;
    b = (1.f + eta) * a.weight;
  }
  __device__ __forceinline__ int row(const Args &, const Place &p, int s) const { return int(p.pos(s)); }

  __device__ __forceinline__ uint32_t address(int s, int k) const {
    return __builtin_amdgcn_perm(w[s][k / 4], low, 0x0c0c0000u | (4u + (k & 3)) << 8);
  }
  // sum_j (z_j - z_i) on the tile at offset IN: the neighbours pairwise, so that DEG equal values sum exactly and
  // cancel DEG * z exactly
  template <uint32_t IN>
  __device__ __forceinline__ f4 diff_sum(int s, f4 z) const {
    auto nb = [&](int k) { return lds_read(address(s, k) + IN); };
    f4 sum;
    if constexpr (DEG == 2) sum = nb(0) + nb(1);
    else if constexpr (DEG == 4) sum = (nb(0) + nb(2)) + (nb(1) + nb(3));
    else sum = ((nb(0) + nb(4)) + (nb(2) + nb(6))) + ((nb(1) + nb(5)) + (nb(3) + nb(7)));
    return fma4(-float(DEG), z, sum);
  }
  __device__ __forceinline__ float scale() const { return b; }
  // sum_j W_ji (z_j - z_i) of a plain round (eta = 0) on the tile at offset 0, term by term in the order of the list.  The
  // pairwise sum above rounds at DEG times the magnitude of z: not where its result is the step itself.
  __device__ __forceinline__ f4 plain(int s, f4 z) const {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < DEG; ++k) acc = fma4(b, lds_read(address(s, k)) - z, acc);
    return acc;
  }
  // The table's registers are made opaque once per round: otherwise the addresses, 4 DEG of them, are computed ahead
  // of the round loop and kept, in four times the registers.
  __device__ __forceinline__ void keep_packed() {
    if constexpr (S == kSlotsMax) {
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int q = 0; q < kWords; ++q) asm volatile("" : "+v"(w[s][q]));
    }
  }
};

// One weight, at most 8 neighbours, more than 256 workers: as ByteRounds with two bytes to a neighbour, the LDS offset of
// its row, 16 bits of which name any row of a tile.  An address costs the same one instruction, the table DEG/2 registers a
// row; against the lists in LDS a round saves a read in three and half of the instructions (300 workers, 4-regular, d =
// 100,000, K = 8: phase 314 -> 257 us; 600 workers, d = 50,000, K = 4 304 -> 240; ring of 1000, d = 60,000, bf16 state,
// K = 4, Algorithm 2's phase 541 -> 297).
struct HalfArgs {
  const uint32_t *offsets;  // DEG / 2 words per position
  float weight;
};
template <int DEG>
struct HalfRounds {
  static constexpr int kSlots = kSlotsMax, kParked = 1, kWaves = DEG <= 4 ? 6 : 5, kWords = DEG / 2;
  static constexpr bool kRowsInMemory = false;
  using Args = HalfArgs;
  uint32_t w[kSlots][kWords];
  float b;

  __device__ __forceinline__ void fetch(const Args &, const Place &) {}
  __device__ __forceinline__ void init(const Args &a, const Place &p, float eta) {
    const uint32_t col_bytes = p.col() * 4u;
#pragma unroll
    for (int s = 0; s < kSlots; ++s)
#pragma unroll
      for (int q = 0; q < kWords; ++q) w[s][q] = a.offsets[p.pos(s) * kWords + q] + col_bytes * 0x00010001u;
    b = (1.f + eta) * a.weight;
  }
  __device__ __forceinline__ int row(const Args &, const Place &p, int s) const { return int(p.pos(s)); }

  __device__ __forceinline__ f4 neighbour(int s, int k) const {
    return lds_read(k & 1 ? w[s][k / 2] >> 16 : w[s][k / 2] & 0xffffu);
  }
  // Difference by difference, pairwise.  The sum of the neighbours, rounded at DEG times the magnitude of z, would take
  // three instructions less of nine and leave a quarter more error against 64 bits than the lists in LDS (300 workers,
  // 4-regular, K = 8: 5.8e-8 against 4.6e-8; so 4.6e-8).
  template <uint32_t IN>
  __device__ __forceinline__ f4 diff_sum(int s, f4 z) const {
    static_assert(IN == 0, "one tile");
    f4 d[DEG];
#pragma unroll
    for (int k = 0; k < DEG; ++k) d[k] = neighbour(s, k) - z;
#pragma unroll
    for (int o = DEG / 2; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) d[k] += d[k + o];
    return d[0];
  }
  __device__ __forceinline__ float scale() const { return b; }
  __device__ __forceinline__ f4 plain(int s, f4 z) const {  // as in ByteRounds
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < DEG; ++k) acc = fma4(b, neighbour(s, k) - z, acc);
    return acc;
  }
  __device__ __forceinline__ void keep_packed() {
#pragma unroll
    for (int s = 0; s < kSlots; ++s)
#pragma unroll
      for (int q = 0; q < kWords; ++q) asm volatile("" : "+v"(w[s][q]));
  }
};

// The lists of a context, laid out for its geometry.
struct ListArgs {
  // 4 * threads / lanes-per-row positions: row number of each (-1: none)
  const int32_t *rows;
  // per (wavefront, slot): first pair of its lists (pairs of all its rows are interleaved), pairs per row
  const uint32_t *groups;
  // the lists: {offset 0, weight 0, offset 1, weight 1}; offsets are LDS byte offsets of rows
  const f4 *pairs;
  int pair_count;       // 16-byte words in `pairs`
  uint32_t tile_bytes;  // where CsrRounds keeps the lists in LDS
};

template <int S>
struct CsrRounds {
  static constexpr int kSlots = S, kWaves = S == 4 ? 6 : 4, kParked = 0;
  static constexpr bool kRowsInMemory = true;
  using Args = ListArgs;
  uint32_t first[S], count[S];  // uniform in a wavefront
  uint32_t list;                // LDS offset of the lane's row in a group's first pair
  uint32_t col_bytes, step;
  float cm;

  __device__ __forceinline__ void fetch(const Args &, const Place &) {}
  __device__ __forceinline__ void init(const Args &a, const Place &p, float eta) {
    for (int k = int(p.tid); k < a.pair_count; k += int(p.threads)) lds_write(a.tile_bytes + 16u * k, a.pairs[k]);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(p.tid >> 6), rows_per_wave = 64u >> p.lpr_log2;
#pragma unroll
    for (int s = 0; s < S; ++s) first[s] = a.groups[2 * (wave * S + s)], count[s] = a.groups[2 * (wave * S + s) + 1];
    step = 16u * rows_per_wave;
    list = a.tile_bytes + 16u * ((p.tid & 63u) >> p.lpr_log2);
    col_bytes = p.col() * 4u;
    cm = 1.f + eta;
  }
  __device__ __forceinline__ int row(const Args &a, const Place &p, int s) const { return a.rows[p.pos(s)]; }

  // sum_j W_ji (z_j - z_i); lists are padded to an even length with the row itself, weight 0
  template <uint32_t IN>
  __device__ __forceinline__ f4 diff_sum(int s, f4 z) const {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    uint32_t at = list + first[s] * 16u;
    for (uint32_t k = 0; k < count[s]; ++k, at += step) {
      const f4 e = lds_read(at);
      const f4 n0 = lds_read(__float_as_uint(e[0]) + col_bytes + IN), n1 = lds_read(__float_as_uint(e[2]) + col_bytes + IN);
      acc = fma4(e[1], n0 - z, acc);
      acc = fma4(e[3], n1 - z, acc);
    }
    return acc;
  }
  __device__ __forceinline__ float scale() const { return cm; }
  __device__ __forceinline__ f4 plain(int s, f4 z) const { return diff_sum<0u>(s, z); }  // as in ByteRounds
  __device__ __forceinline__ void keep_packed() { asm volatile("" : "+v"(list), "+v"(col_bytes)); }
};

// The same lists held in registers: at most kListPairs pairs per row.
constexpr int kListPairs = 4;
template <int S>
struct ListRounds {
  static constexpr int kSlots = S, kWaves = 4, kParked = 0;
  static constexpr bool kRowsInMemory = false;
  using Args = ListArgs;
  f4 list[S][kListPairs];
  uint32_t at[S][2 * kListPairs];
  float weight[S][2 * kListPairs];
  int rows[S], pairs[S];  // pairs: uniform in a wavefront
  float cm;

  __device__ __forceinline__ void fetch(const Args &a, const Place &p) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(p.tid >> 6), rows_per_wave = 64u >> p.lpr_log2;
    const uint32_t in_wave = (p.tid & 63u) >> p.lpr_log2;
    uint32_t first[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      rows[s] = a.rows[p.pos(s)];
      first[s] = a.groups[2 * (wave * S + s)], pairs[s] = int(a.groups[2 * (wave * S + s) + 1]);
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int q = 0; q < kListPairs; ++q)
        if (q < pairs[s]) list[s][q] = a.pairs[first[s] + q * rows_per_wave + in_wave];
  }
  __device__ __forceinline__ void init(const Args &, const Place &p, float eta) {
    const uint32_t col_bytes = p.col() * 4u;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int q = 0; q < kListPairs; ++q) {
        // past the end of the list: the row itself with weight 0, so that nobody else's infinity gets in
        at[s][2 * q] = at[s][2 * q + 1] = p.own(s), weight[s][2 * q] = weight[s][2 * q + 1] = 0.f;
        if (q < pairs[s]) {
          const f4 e = list[s][q];
          at[s][2 * q] = __float_as_uint(e[0]) + col_bytes, weight[s][2 * q] = e[1];
          at[s][2 * q + 1] = __float_as_uint(e[2]) + col_bytes, weight[s][2 * q + 1] = e[3];
        }
      }
    cm = 1.f + eta;
  }
  __device__ __forceinline__ int row(const Args &, const Place &, int s) const { return rows[s]; }

  template <uint32_t IN>
  __device__ __forceinline__ f4 diff_sum(int s, f4 z) const {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    auto pair = [&](int q) {
      const f4 n0 = lds_read(at[s][2 * q] + IN), n1 = lds_read(at[s][2 * q + 1] + IN);
      acc = fma4(weight[s][2 * q], n0 - z, acc);
      acc = fma4(weight[s][2 * q + 1], n1 - z, acc);
    };
    // all reads of a list are in flight together; the lists of a wavefront's rows are about as long as each other
    if (pairs[s] <= 2) {
      pair(0), pair(1);
    } else {
      pair(0), pair(1), pair(2), pair(3);
    }
    return acc;
  }
  __device__ __forceinline__ float scale() const { return cm; }
  __device__ __forceinline__ f4 plain(int s, f4 z) const { return diff_sum<0u>(s, z); }  // as in ByteRounds
  __device__ __forceinline__ void keep_packed() {}
};

// The second array of a phase, which waits while the first runs its rounds.  The last kParked of the lane's rows
// wait in LDS behind the tile (16 bytes per lane and row; a lane reads back what it wrote, so there is no barrier).
template <class R>
struct Waiting {
  static constexpr int kHeld = R::kSlots - R::kParked;
  f4 v[kHeld];
  __device__ __forceinline__ void put(const Place &p, int s, f4 x) {
    if (s < kHeld) v[s] = x;
    else lds_write(p.own(s + R::kParked), x);
  }
  __device__ __forceinline__ f4 get(const Place &p, int s) const {
    return s < kHeld ? v[s] : lds_read(p.own(s + R::kParked));
  }
};

// One round: z_r of all rows is in the tile at IN, z_{r+1} goes to the one at OUT.
template <uint32_t IN, uint32_t OUT, class R>
__device__ __forceinline__ void round_step(f4 (&z)[R::kSlots], f4 (&u)[R::kSlots], R &rounds, Place &p, float c, float eta) {
  constexpr int S = R::kSlots;
  rounds.keep_packed();
  if constexpr (S == kSlotsMax) p.forget();
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const f4 t = rounds.template diff_sum<IN>(s, z[s]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float ue = u[s][e];
      fused::momentum(ue, eta, t[e]);
      u[s][e] = ue;
    }
    if constexpr (S == kSlotsMax) __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (IN == OUT) __syncthreads();  // every read of z_r is done
#pragma unroll
  for (int s = 0; s < S; ++s) {
    z[s] = fma4(c, u[s], z[s]);
    lds_write(p.own(s) + OUT, z[s]);
  }
  __syncthreads();  // z_{r+1} is visible (and with two tiles, every read of z_r is done)
}

// K >= 1 rounds from z_{-1} = z_0 = z.  Result in z; u is scratch: the velocity divided by scale(), which takes one
// multiplication per output and round out.
template <class R>
__device__ __forceinline__ void gossip(f4 (&z)[R::kSlots], R &rounds, Place &p, float eta, int K) {
  constexpr int S = R::kSlots;
  f4 u[S];
  p.forget();
#pragma unroll
  for (int s = 0; s < S; ++s) lds_write(p.own(s), z[s]), u[s] = f4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  const float c = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rounds.scale())));
  if constexpr (S == kSlotsMax) {
    for (int r = 0; r < K; ++r) round_step<0u, 0u>(z, u, rounds, p, c, eta);
  } else {
    constexpr uint32_t kSecond = second_tile(S);
    int r = 0;
    for (; r + 2 <= K; r += 2) {
      round_step<0u, kSecond>(z, u, rounds, p, c, eta);
      round_step<kSecond, 0u>(z, u, rounds, p, c, eta);
    }
    if (r < K) {
      round_step<0u, kSecond>(z, u, rounds, p, c, eta);
      // the next use of the first tile starts with writes to it; its last readers passed the barrier above
    }
  }
  p.forget();
}

// Calls request(tile, s, row offset, columns, row) for the lane's rows in turn and, AHEAD rows behind, use(tile, s, row offset,
// columns, mine, what request returned), with the scheduler fenced in between: left alone, the compiler issues every row's
// loads at once and spills.  (kInOneGo: both between the same two fences.)  `tile` is a compile-time value of Tile.  A position
// past the last row reads row 0 and must not store (mine = false); no list names it.  CUT as above.
template <int AHEAD, class R, bool CUT, class Request, class Use>
__device__ __forceinline__ void each_row(const R &rounds, const typename R::Args &ra, Place &p, int tile, int n, int64_t d,
                                         int64_t ld, int64_t first, Request &&request, Use &&use) {
  constexpr int S = R::kSlots;
  int rows[S];
  if constexpr (R::kRowsInMemory) {  // together, and not each ahead of its own accesses
    p.forget();
#pragma unroll
    for (int s = 0; s < S; ++s) rows[s] = rounds.row(ra, p, s);
    __builtin_amdgcn_sched_barrier(0);
  }
  auto go = [&](auto of) {
    if constexpr (AHEAD == kInOneGo) {  // as below, but written out: through a function ByteRounds spill 2 to 4 registers more
#pragma unroll
      for (int s = 0; s < S; ++s) {
        p.forget();
        Columns c{first + p.col(), 0};
        if (of == kCut && c.at > d - 4) c = Columns{d - 4, int(c.at - (d - 4))};
        const int row = R::kRowsInMemory ? rows[s] : rounds.row(ra, p, s);
        const bool mine = row >= 0 && row < n;
        const int64_t off = int64_t(mine ? row : 0) * ld;
        use(of, s, off, c, mine, request(of, s, off, c, row));
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    auto at = [&](int s, auto &&f) {
      p.forget();
      Columns c{first + p.col(), 0};
      if (of == kCut && c.at > d - 4) c = Columns{d - 4, int(c.at - (d - 4))};
      const int row = R::kRowsInMemory ? rows[s] : rounds.row(ra, p, s);
      const bool mine = row >= 0 && row < n;
      f(int64_t(mine ? row : 0) * ld, c, row, mine);
      __builtin_amdgcn_sched_barrier(0);
    };
    decltype(request(of, 0, int64_t{}, Columns{}, 0)) on_the_way[S];
#pragma unroll
    for (int s = 0; s < S + AHEAD; ++s) {
      if (s < S) at(s, [&](int64_t off, Columns c, int row, bool) { on_the_way[s] = request(of, s, off, c, row); });
      if (s >= AHEAD)
        at(s - AHEAD, [&](int64_t off, Columns c, int, bool mine) { use(of, s - AHEAD, off, c, mine, on_the_way[s - AHEAD]); });
    }
  };
  if (tile >= kWhole) {
    go(std::integral_constant<int, kWhole>{});
  } else {
    if (CUT && tile == kCut) go(std::integral_constant<int, CUT ? kCut : kNarrow>{});
    else go(std::integral_constant<int, kNarrow>{});
  }
}
// use(tile, s, row offset, columns, mine) alone.
struct Nothing {};
template <class R, bool CUT, class Use>
__device__ __forceinline__ void each_row(const R &rounds, const typename R::Args &ra, Place &p, int tile, int n, int64_t d,
                                         int64_t ld, int64_t first, Use &&use) {
  each_row<kInOneGo, R, CUT>(rounds, ra, p, tile, n, d, ld, first, [&](auto, int, int64_t, Columns, int) { return Nothing{}; },
                             [&](auto F, int s, int64_t off, Columns c, bool mine, Nothing) { use(F, s, off, c, mine); });
}

// Columns, rows per lane and threads of a block.  A tile takes 16 bytes per lane and row: 64 KiB at most.
struct Geometry {
  int cols = 0, slots = 0, threads = 0;
  int lpr_log2() const { return __builtin_ctz(unsigned(cols)) - 2; }
  int positions() const { return slots * threads / (cols / 4); }
  // LDS without lists: the tile and the parked rows, or two tiles
  size_t tile_bytes(int parked) const {
    return slots < kSlotsMax ? second_tile(slots) + size_t(slots) * threads * 16 : size_t(slots + parked) * threads * 16;
  }
};

inline Geometry geometry_for(int n, int cols, int slots) {
  Geometry g;
  const int lanes = (n + slots - 1) / slots * (cols / 4), threads = (lanes + 63) / 64 * 64;
  if (threads <= kThreadsMax) g.cols = cols, g.slots = slots, g.threads = threads;
  return g;
}

constexpr int kByteRows = 256;                 // rows a one-byte table can name
constexpr size_t kLdsMax = size_t(160) << 10;  // LDS of a compute unit

// A matrix is small while one row per lane leaves it no more wavefronts than the chip runs at a time (256 compute units
// x 32 wavefronts of 64 lanes x 4 columns: 2 Mi elements).  Measured per step, K = 12, fp32, one row or two per lane
// against four: n = 64, d = 16,000 10.6 against 21.8 us (10.6 is what a call takes the host), n = 12 irregular,
// d = 64,000 12.8 against 39 us; from 3 Mi elements on four rows are as fast or faster (n = 48, d = 64,000, K = 2: 19
// against 22 us).
inline bool small_matrix(int n, int64_t d) { return int64_t(n) * ((d + 3) / 4) <= int64_t(8192) * 64; }

// A small matrix: the fewest rows per lane with which a tile of at most 64 columns fits a block.  cols = 0: none does.
inline Geometry small_geometry(int n, int cols_min) {
  Geometry g;
  for (int slots = 1; slots < kSlotsMax; slots *= 2)
    for (int cols = 64; cols >= cols_min; cols /= 2) {
      g = geometry_for(n, cols, slots);
      if (g.cols) return g;
    }
  return g;
}

// Four rows per lane: as wide a tile as a block of about 256 threads holds, between 64 and 256 columns: several small
// blocks on a compute unit drift apart and keep memory and LDS busy at once, where two blocks of 1024 threads tend to
// load and to compute in turn (64 Mi elements, fp32, 4-regular, K = 8, tile of 64 / 128 / 256 columns: n = 64 331 /
// 333 / 380 us, n = 128 385 / 458 us, n = 24 374 / 329 / 354 us).  Tiles of 32 columns for n > 128 (an instruction more
// per address, row pieces of 64 to 128 bytes) measured slower (n = 256, bf16 state, K = 8: 457 against 417 us).  5 to 8
// workers take 128 columns, which makes a block one wavefront (against 256: 1 % faster in the median of n = 5 ... 8, both
// state types, 3 to 100 Mi elements, K = 1 and 8; 5 to 10 % at K = 8 and 100 Mi, up to 6 % slower at K = 1 and 3 Mi).
inline Geometry byte_geometry(int n, int64_t d) {
  Geometry g;
  if (small_matrix(n, d)) {
    g = small_geometry(n, 64);
    if (g.cols) return g;
  }
  for (int cols = n > 4 && n <= 8 ? 128 : 256; cols >= 64; cols /= 2) {
    g = geometry_for(n, cols, kSlotsMax);
    if (g.cols && g.threads <= 320) break;
  }
  return g;
}

// The same for the lists, which go down to 32 columns (n = 100 610 against 681 us with 64, n = 256 647 against 793 us)
// and to 16 where a tile of 32 does not fit a block.  cols = 0: n does not fit.
inline Geometry csr_geometry(int n, int64_t d) {
  Geometry g;
  if (small_matrix(n, d)) {
    g = small_geometry(n, 16);
    if (g.cols) return g;
  }
  for (int cols = 256; cols >= 16; cols /= 2) {
    g = geometry_for(n, cols, kSlotsMax);
    if (g.cols && (g.threads <= 256 || cols == 32)) break;
  }
  return g;
}

// A launch that asks for more LDS than the default limit raises it for its kernel first, always to the same value: the
// limit is the process's, and contexts on other host threads launch the same kernel with lists of another length.
inline int allow_lds(const void *kernel, size_t bytes) {
  if (bytes <= 65536) return 0;
  return hip_rc(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsMax)));
}

enum Call : int { kPlain, kAtc, kFusedStep, kAlg2, kDpsgd };  // the last three read a matrix late

// How a call of tiles that share cache lines (rows that do not start on one, or tiles of 32 columns of bf16 state) treats
// them: up to `reads` MiB only its stores stream, from there to `streams` MiB all does, beyond nothing.  A shared line that
// streams is gone before the other tile wants it, or goes to memory half written; the wider the tile, the fewer are shared.
// Streamed, loads kept, all kept, K = 4, three states in turn:
// Up to 64 columns every other line is shared and nothing that streams does well: phase, 64 x 1,000,001 481, 382, 337 us,
// fused step 637, 453, 401, bf16 540, 354, 301; up to 192 MiB of rows of 256 bytes and more the stores may: fused step 64 x
// 100,001 58, 41, 44.
// 128 columns (5 to 8 and 21 to 40 workers): fused step, n = 28, 200 MiB 99, 88, 89, 330 MiB 174, 143, 138; ATC phase, n =
// 40, 200 MiB 82, 81, 86, 420 MiB 172, 159, 156; D-PSGD 330 MiB 126, 116, 113.
// 256 columns (up to 20 workers): ATC phase, n = 20, 128 MiB 48.9, 48.2, 53.8, 200 MiB 75, 80, 83, 330 MiB 114, 120, 122, 560
// MiB 201, 199, 199; fused step, n = 12, 260 MiB 111, 105, 109, 560 MiB 242, 223, 220; D-PSGD 128 MiB 38.8, 36.1, 41.1, 200
// MiB 61, 65, 67, 420 MiB 139, 138, 137.  With up to 4 rows a tile the loads are best kept: ATC phase, n = 3, 210 MiB 75, 72,
// 78.
// Plain gossip of lists: n = 16, 260 MiB 130, 144, 144, n = 24 (128 columns) 180 MiB 101, 104, 101; of bf16 state: n = 20, 160
// MiB 115, 122, 122, n = 28 128 MiB 91, 95, 94, 200 MiB 147, 148, 146.
struct SharedLines {
  int reads, streams;
};
inline SharedLines shared_lines(const Shape &s, const Geometry &g, Call call, bool lists) {
  constexpr int kEver = 1 << 30;
  if (g.cols < 128) return g.cols * (s.bf16 ? 2 : 4) >= 256 ? SharedLines{192, 192} : SharedLines{0, 0};
  const bool wide = g.cols > 128;
  if (call == kPlain) {
    if (wide && (lists || s.bf16)) return {96, kEver};
    if (lists) return {96, 96};
    if (s.bf16) return {100, 176};
  }
  if (wide && s.n <= 4) return {400, 400};
  switch (call) {
    case kAtc: return wide ? SharedLines{144, 480} : SharedLines{260, 260};
    case kFusedStep: return wide ? SharedLines{288, 288} : SharedLines{260, 260};
    case kDpsgd: return wide ? SharedLines{144, 300} : SharedLines{192, 192};
    default: return {192, 192};
  }
}

// How these kernels treat the caches: calls f(access).  Matrices with S < 4 fit the caches.
// Where tiles have their cache lines to themselves a call streams; up to 128 MiB the calls that read a matrix late (the
// gradients of Algorithm 2's phase and of D-PSGD, the old gradient of the fused step) leave the loads to the caches.
// Streamed, loads kept, all kept, K = 4, three states in turn: Algorithm 2's phase 64 x 100,001 34.3, 32.2, 31.7 us, 20 x
// 200,001 22.8, 20.2, 19.1; fused step 20 x 200,001 27.9, 25.7, 26.3, 64 x 200,001 78.9, 82.1, 85.2; but the ATC phase
// 64 x 50,001 21.4, 22.0, 22.9, 256 x 30,001 40.2, 40.3, 46.9.  Plain gossip of up to 32 MiB streams wherever its rows start:
// 64 x 50,001 9.7, 10.6, 10.4 us.
template <class R, class F>
int with_access(const Shape &s, const Geometry &g, Call call, int per_element, std::initializer_list<const void *> matrices,
                F &&f) {
  if constexpr (R::kSlots < kSlotsMax) {
    return f(AccessTag<kKeepReads>{});
  } else {
    const int64_t mib = fused::footprint(s, per_element) >> 20;
    if (call == kPlain && mib < 32) return f(AccessTag<kStream>{});
    SharedLines lines{call > kAtc ? 128 : 0, 1 << 30};
    if (fused::shares_lines(s, matrices) || g.cols * (s.bf16 ? 2 : 4) % 128 != 0)
      lines = shared_lines(s, g, call, std::is_same_v<typename R::Args, ListArgs>);
    if (mib < lines.reads) return f(AccessTag<kKeepReads>{});
    return mib < lines.streams ? f(AccessTag<kStream>{}) : f(AccessTag<kKeep>{});
  }
}

template <class R>
struct RoundsTag {
  using type = R;
};

// Calls f(RoundsTag<R>, geometry, LDS bytes, R::Args) for the table's form and the shape's geometry.
template <class F>
int with_rounds(const Shape &s, const LdsTable &t, F &&f) {
  if (t.bytes_deg) {
    const Geometry g = byte_geometry(s.n, s.d);
    auto go = [&](auto r) {
      using R = typename decltype(r)::type;
      return f(r, g, g.tile_bytes(R::kParked), typename R::Args{t.byte_table, t.weight});
    };
    auto with_degree = [&](auto slots) {
      constexpr int S = decltype(slots)::value;
      switch (t.bytes_deg) {
        case 2: return go(RoundsTag<ByteRounds<2, S>>{});
        case 4: return go(RoundsTag<ByteRounds<4, S>>{});
        default: return go(RoundsTag<ByteRounds<8, S>>{});
      }
    };
    return g.slots == 1   ? with_degree(std::integral_constant<int, 1>{})
           : g.slots == 2 ? with_degree(std::integral_constant<int, 2>{})
                          : with_degree(std::integral_constant<int, 4>{});
  }
  if (!t.pairs && !t.half_deg) return -1;
  const Geometry g = csr_geometry(s.n, s.d);
  if (t.half_deg) {
    auto go = [&](auto r) {
      using R = typename decltype(r)::type;
      return f(r, g, g.tile_bytes(R::kParked), HalfArgs{t.offsets, t.weight});
    };
    switch (t.half_deg) {
      case 2: return go(RoundsTag<HalfRounds<2>>{});
      case 4: return go(RoundsTag<HalfRounds<4>>{});
      default: return go(RoundsTag<HalfRounds<8>>{});
    }
  }
  auto go = [&](auto r) {
    using R = typename decltype(r)::type;
    const size_t tile = g.tile_bytes(R::kParked), lists = t.max_pairs <= kListPairs && R::kSlots < kSlotsMax ? 0 : t.pair_count;
    return f(r, g, tile + lists * 16,
             ListArgs{t.rows, t.groups, reinterpret_cast<const f4 *>(t.pairs), t.pair_count, uint32_t(tile)});
  };
  const bool in_registers = t.max_pairs <= kListPairs;
  switch (g.slots) {
    case 1: return in_registers ? go(RoundsTag<ListRounds<1>>{}) : go(RoundsTag<CsrRounds<1>>{});
    case 2: return in_registers ? go(RoundsTag<ListRounds<2>>{}) : go(RoundsTag<CsrRounds<2>>{});
    default: return go(RoundsTag<CsrRounds<4>>{});
  }
}

}  // namespace lds_tile
}  // namespace detag
