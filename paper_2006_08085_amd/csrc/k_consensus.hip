// The whole factor sequence of the exact average consensus (Lemma 1 of the
// paper; spanning-tree gather and propagate steps) applied on chip, for up to
// 256 workers: Z <- A_{R-1} ... A_0 Z with the state read and written once.
//
// A wavefront owns 32 columns (more with few workers) and all n rows of them; the rows sit in LDS (128
// bytes each) and stay there.  A gather or propagate step changes only the rows
// of one level of the tree and their parents; every other row of the factor is
// an identity row and costs nothing, and a changed row that no later step reads
// before it is overwritten again (the emptied rows of the gather steps) is
// dropped on the host.  What remains is a list of row operations
//   row[dst] = sum_k w_k * row[o_k],   at most 8 terms,
// to be done in order; the host packs them, eight at a time, into groups that
// may be done side by side: no row of a group is read by a later row of it, so
// that the order within a group does not matter once every operand is read
// before any row is written.  Rows of different steps share a group where
// nothing forbids it, which makes the number of groups little more than the
// depth of the tree: 64 workers, 4-regular: 15 groups, 22 slots of two terms
// (batches of four operations within a step: 42).
//
// Eight lanes side by side take a row, four columns each, and the eight rows of
// a group are done at once: a slot of two terms is two 16-byte LDS reads, eight
// multiply-adds and, after the last slot of a group, one 16-byte write, with the
// operands of a lane's row in one 16-byte word fetched some slots ahead.  An
// absent term reads a row of zeros with weight 0, an idle lane writes to it.  No
// wavefront waits for another: there is no barrier.
//
// With one column per lane, the four operations of a batch one after the other
// and 16 KiB of LDS per wavefront (10 of them on a compute unit, 19 now), 64
// workers, 4-regular, d = 272,474 took 49 us, 31 now; d = 1,000,000 139 and 109;
// 256 workers, d = 400,000 566 and 257; 64 workers, d = 20,000 14.5 and 6.8.
//
// The words of the slots come through vector memory, where they queue behind the
// rows of other wavefronts: 16 workers, bf16 state, 300 MiB 207 us, where one
// column per lane and words in scalar registers had taken 184.  A tile of few
// workers leaves room in LDS for a copy of them per wavefront: 164 us.
#include <algorithm>

#include "detag_internal.h"
#include "dev_common.hpp"
#include "fused_common.hpp"
#include "fused_generic_common.hpp"

namespace detag {
namespace {

using namespace lds_tile;

constexpr int kRowsMax = 256, kTerms = 8;
constexpr int kProgramRow = 256;  // bytes per row index in the program that detag_factors_get_program shows
constexpr int kBatch = 4;         // its operations per batch

struct Op {
  uint32_t o0, o1, dst;  // byte offsets of the two source rows and of the written row in the tile (< 65536)
  uint32_t keep;         // all ones: continue the previous operation's sum; 0: start from 0
  uint32_t w0, w1;       // fp32 weights
  uint32_t m0, m1;       // all ones: the term is there; 0: it is not
};
constexpr int kOpWords = sizeof(Op) / 4;

// Lanes side by side that take a row.  Few workers make few rows that can be done side by side and a tile that is soon
// loaded: wider rows keep the wavefronts busy, and their pieces of a row fill the cache lines, until the tiles leave too few
// wavefronts on a compute unit (8, 16 and 32 lanes; fp32 unless said otherwise, 4-regular: n = 8, 300 MiB of bf16 -, 171,
// 142 us; n = 12, 64 MiB of bf16 -, 38, 34, 300 MiB -, 158, 180; n = 16, 4 MiB -, 5.8, 6.6, 300 MiB -, 125, 125, of a ring -,
// 132, 126; n = 24, 300 MiB 129, 126, -; n = 28, 24 MiB 12.3, 11.1, -, 160 MiB 75, 68, -, of bf16 64 MiB 41, 37, -, 160 MiB
// 126, 108, -; n = 32, 64 MiB of bf16 36, 40, -, 300 MiB 216, 216, -; n = 40, 160 MiB 77, 70, -; ring of 48, 300 MiB 171, 142,
// 163; n = 64, 64 MiB 29, 32, 38).
int lanes_per_row(const Shape &s) {
  const int64_t mib = fused::footprint(s, s.bf16 ? 2 : 4) >> 20;
  if (s.bf16) return s.n <= 8 || (s.n <= 12 && mib < 88) ? 32 : s.n <= 24 || (s.n <= 32 && mib >= 88) ? 16 : 8;
  const int narrow = mib >= 256 ? 48 : mib >= 128 ? 40 : mib >= 16 ? 32 : 24;  // up to here, 16 lanes
  return s.n <= (mib >= 16 ? 16 : 12) ? 32 : s.n <= narrow ? 16 : 8;
}
// Whether each wavefront has a copy of its table behind the tiles.  It pays while wavefronts enough remain (table in memory
// and in LDS, 300 MiB: fp32 n = 16 131 and 125 us, 32 135 and 133, 40 133 and 127; bf16 n = 8 184 and 142, 16 207 and 164, 20
// 179 and 157, but n = 12 in rows of 32 lanes 64 MiB 34 and 36, ring of 24 221 and 243); a long one only where the rows crowd
// vector memory (bf16, ring of 16 64 MiB 41 and 42, 88 MiB 68 and 62), and small calls do without (fp32 n = 24, 4 MiB 5.0 and
// 5.4; bf16 n = 16, 20 MiB 16.2 and 17.0).
bool table_in_lds(const Shape &s, size_t tile_bytes, size_t table_bytes) {
  const int lanes = lanes_per_row(s);
  const int64_t mib = fused::footprint(s, s.bf16 ? 2 : 4) >> 20;
  if (lanes == 8 || mib < (s.bf16 && lanes == 16 ? 32 : 16) || (s.bf16 && s.n > (lanes == 32 ? 8 : 20))) return false;
  return table_bytes * 4 <= tile_bytes || mib >= (s.bf16 ? 88 : 80);
}
template <int LPR>
struct Layout {
  static constexpr int kCols = 4 * LPR, kGroup = 64 / LPR;  // columns of a wavefront, rows done side by side
  static constexpr uint32_t kRowBytes = kCols * 4;
};
constexpr int kSlotsPadded = 4;  // the number of slots is a multiple of it
constexpr int kChunk = 8;        // rows a lane loads or stores together

// What a row of a group does in a slot: the LDS offsets of two source rows (the second in the upper half of the word), the
// offset of the written row with kLast in the group's last slot, two fp32 weights.
struct alignas(16) Entry {
  uint32_t from, to;
  float w0, w1;
};
constexpr uint32_t kLast = 1u << 16;

template <typename ST, int LPR, bool TABLE_IN_LDS, Access A>
__global__ __launch_bounds__(256, TABLE_IN_LDS ? 8 : 7) void factor_sequence_kernel(ST *Z, int n, int64_t d, int64_t ld,
                                                                                 const Entry *__restrict__ table, int slots) {
  constexpr int kAhead = TABLE_IN_LDS ? 2 : kSlotsPadded;
  constexpr int kCols = Layout<LPR>::kCols, kGroup = Layout<LPR>::kGroup;
  constexpr uint32_t kRowBytes = Layout<LPR>::kRowBytes;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  uint32_t group = lane / LPR;
  // neighbouring tiles on one XCD (64 x 3,000,000 542 -> 493 us, odd pitch 64 x 300,007 68 -> 59 us)
  const int64_t first = (fused::xcd_tile(blockIdx.x, gridDim.x) * (blockDim.x >> 6) + w) * kCols;
  if (first >= d) return;  // no barrier anywhere below
  const uint32_t tile = w * uint32_t(n + 1) * kRowBytes + (lane % LPR) * 16u;  // the lane's columns of row 0
  const uint32_t copy = (blockDim.x >> 6) * uint32_t(n + 1) * kRowBytes + w * uint32_t(slots) * (kGroup * 16u);
  auto entry = [&](int slot) {
    if constexpr (TABLE_IN_LDS) return __builtin_bit_cast(Entry, lds_read(copy + (slot * kGroup + lane / LPR) * 16u));
    else return table[slot * kGroup + lane / LPR];
  };
  Entry ahead[kAhead];
  auto fetch_first = [&] {
#pragma unroll
    for (int q = 0; q < kAhead; ++q) ahead[q] = entry(q);
  };
  if constexpr (TABLE_IN_LDS) {
    for (int q = int(lane); q < slots * kGroup; q += 64) lds_write(copy + q * 16u, *reinterpret_cast<const f4 *>(table + q));
  } else {
    fetch_first();
  }
  Columns c{first + (lane % LPR) * 4, 0};
  const int kind = d - first >= kCols ? kWhole : d - first >= 4 ? kCut : kNarrow;
  if (kind == kCut && c.at > d - 4) c = Columns{d - 4, int(c.at - (d - 4))};
  // f(kind, k, row) for the lane's rows of a chunk; past the last row it is repeated, which does no harm
  auto each_row = [&](int r0, auto of, auto f) {
    asm volatile("" : "+v"(group));  // addresses are made anew, not kept
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (r0 + k * kGroup < n) f(of, k, min(r0 + k * kGroup + int(group), n - 1));
  };
  auto with_kind = [&](auto f) {
    if (kind == kWhole) f(std::integral_constant<int, kWhole>{});
    else if (kind == kCut) f(std::integral_constant<int, kCut>{});
    else f(std::integral_constant<int, kNarrow>{});
  };
  if (group == 0) lds_write(tile + uint32_t(n) * kRowBytes, f4{0.f, 0.f, 0.f, 0.f});
  with_kind([&](auto kind_of) {
    for (int r0 = 0; r0 < n; r0 += kChunk * kGroup) {
      Raw<ST> v[kChunk];
      each_row(r0, kind_of, [&](auto of, int k, int row) { v[k] = load4<of, A>(Z, int64_t(row) * ld, c, d); });
      __builtin_amdgcn_sched_barrier(0);
      each_row(r0, kind_of, [&](auto, int k, int row) { lds_write(tile + uint32_t(row) * kRowBytes, floats(v[k])); });
    }
  });
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // lanes read what others wrote
  if constexpr (TABLE_IN_LDS) fetch_first();
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < slots; s += kAhead) {
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const Entry e = ahead[q];
      ahead[q] = entry(s + kAhead < slots ? s + kAhead + q : q);
      acc = fma4(e.w0, lds_read(tile + (e.from & 0xffffu)), acc);
      acc = fma4(e.w1, lds_read(tile + (e.from >> 16)), acc);
      if (__builtin_amdgcn_readfirstlane(e.to) & kLast) {  // the same in all groups
        lds_write(tile + (e.to & 0xffffu), acc);
        acc = f4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  with_kind([&](auto kind_of) {
    for (int r0 = 0; r0 < n; r0 += kChunk * kGroup) {
      f4 v[kChunk];
      each_row(r0, kind_of, [&](auto, int k, int row) { v[k] = lds_read(tile + uint32_t(row) * kRowBytes); });
      __builtin_amdgcn_sched_barrier(0);
      each_row(r0, kind_of, [&](auto of, int k, int row) { store4<of, A>(Z, int64_t(row) * ld, c, d, v[k]); });
    }
  });
}

uint32_t f32_bits(float f) {
  uint32_t u;
  __builtin_memcpy(&u, &f, sizeof u);
  return u;
}

// LDS of a compute unit as far as one block may use it on the current device (queried once).
int max_lds_per_block() {
  static const int bytes = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    return v;
  }();
  return bytes;
}

// How the sequence treats the caches: as the other tile kernels where tiles share cache lines (64 x 1,000,001 streamed,
// loads kept, all kept 249, 155, 131 us).  On lines, sequences that fit the memory-side cache beside other matrices leave
// the loads to it (64 x 272,474 31.5, 30.4, 29.9; 8 x 3,000,000 of bf16 30.7, 25.3, 25.2), small ones with fp32 state do not
// (16 x 272,474 9.9, 11.0, 11.1; with a copy of the table in LDS they do from 26 MiB on, 9 x 850,000 15.3, 13.5, -), large
// ones stream (64 x 1,000,000 109, 117, 118; 16 workers, bf16, 88 MiB 53, 54, 55, 160 MiB 88, 94, 94).  Pieces of half a line
// (8 lanes to a row of bf16) are left to the caches up to 64 workers: 64 workers 24 MiB 24.4, 22.4, 22.3, 88 MiB 73, 74, 72,
// 300 MiB 261, 251, 241, 40 workers 300 MiB 231, 218, 213; but 128 workers 104 MiB 115, 121, 122 and 256 workers 300 MiB 555,
// 590, 599.
Access sequence_access(const Shape &s, const void *Z) {
  if (fused::shares_lines(s, {Z})) return kKeep;
  const int64_t mib = fused::footprint(s, s.bf16 ? 2 : 4) >> 20;
  const bool narrow = lanes_per_row(s) == 8;
  if (s.bf16) return narrow && s.n <= 64 ? kKeep : mib >= (narrow ? 96 : 88) ? kStream : kKeepReads;
  return mib >= 96 || mib < (narrow ? 32 : 26) ? kStream : kKeepReads;
}

struct Row {  // a row of a factor that is not an identity row
  int dst, cnt;
  int col[kTerms];
  float val[kTerms];
};

// Order the changed rows of one step so that whoever reads a row that the step also overwrites comes before (or is)
// the row's writer.  False if they read each other in a cycle.
bool order_rows(int n, std::vector<Row> &rows) {
  const int m = int(rows.size());
  std::vector<int> writer(n, -1), waits(m, 0);
  for (int a = 0; a < m; ++a) writer[rows[a].dst] = a;
  std::vector<std::vector<int>> then(m);  // then[b]: writers that have to come after reader b
  for (int b = 0; b < m; ++b)
    for (int k = 0; k < rows[b].cnt; ++k) {
      const int a = writer[rows[b].col[k]];
      if (a >= 0 && a != b) then[b].push_back(a), ++waits[a];
    }
  std::vector<int> order, ready;
  for (int a = m - 1; a >= 0; --a)
    if (!waits[a]) ready.push_back(a);
  while (!ready.empty()) {
    const int b = ready.back();
    ready.pop_back();
    order.push_back(b);
    for (int a : then[b])
      if (--waits[a] == 0) ready.push_back(a);
  }
  if (int(order.size()) != m) return false;
  std::vector<Row> sorted;
  sorted.reserve(m);
  for (int i : order) sorted.push_back(rows[i]);
  rows.swap(sorted);
  return true;
}

// Drop every changed row whose value nobody uses: going back from the last step, a row is needed after a step if
// it is part of the result or a later kept row reads it before it is written again.
void drop_unused_rows(int n, std::vector<std::vector<Row>> &steps) {
  std::vector<char> needed(n, 1);
  for (size_t s = steps.size(); s-- > 0;) {
    std::vector<Row> kept;
    for (const Row &r : steps[s])
      if (needed[r.dst]) kept.push_back(r);
    for (const Row &r : kept) needed[r.dst] = 0;  // a step reads the state before it, so first the writes...
    for (const Row &r : kept)
      for (int k = 0; k < r.cnt; ++k) needed[r.col[k]] = 1;  // ...then what they read
    steps[s].swap(kept);
  }
}

}  // namespace

// The table is an even number of batches; a batch never holds rows of two steps.
bool build_factor_table(int n, const std::vector<HostFactor> &factors, std::vector<uint32_t> &table) {
  table.clear();
  if (n > kRowsMax) return false;
  std::vector<std::vector<Row>> steps;
  for (const HostFactor &f : factors) {
    std::vector<Row> rows;
    for (int i = 0; i < n; ++i) {
      const int b = f.rowptr[i], cnt = f.rowptr[i + 1] - b;
      if (cnt > kTerms) return false;
      if (cnt == 1 && f.colidx[b] == i && f.vals[b] == 1.0) continue;  // identity row: nothing to do
      Row r{};
      r.dst = i, r.cnt = cnt;
      for (int k = 0; k < cnt; ++k) r.col[k] = f.colidx[b + k], r.val[k] = float(f.vals[b + k]);
      rows.push_back(r);
    }
    steps.push_back(std::move(rows));
  }
  drop_unused_rows(n, steps);
  const auto row_off = [](int i) { return uint32_t(i) * kProgramRow; };
  const uint32_t ones = ~0u, one_f = f32_bits(1.f);
  std::vector<Op> ops;
  for (std::vector<Row> &rows : steps) {
    if (!order_rows(n, rows)) return false;
    int room = 0;  // operations left in the open batch
    const auto close_batch = [&] {  // fill up with operations that write the last sum to its row once more
      for (; room > 0 && !ops.empty(); --room) {
        const Op &last = ops.back();
        ops.push_back(Op{last.dst, last.dst, last.dst, ones, 0u, 0u, 0u, 0u});
      }
    };
    for (const Row &r : rows) {
      const int nops = r.cnt > 2 ? (r.cnt + 1) / 2 : 1;
      if (nops > room) close_batch(), room = kBatch;
      for (int o = 0; o < nops; ++o) {
        const int k0 = 2 * o, terms = r.cnt - k0 >= 2 ? 2 : r.cnt - k0;
        Op op{row_off(r.dst), row_off(r.dst), row_off(r.dst), o > 0 ? ones : 0u, 0u, 0u, 0u, 0u};
        if (terms > 0) op.o0 = row_off(r.col[k0]), op.w0 = f32_bits(r.val[k0]), op.m0 = ones;
        if (terms > 1) op.o1 = row_off(r.col[k0 + 1]), op.w1 = f32_bits(r.val[k0 + 1]), op.m1 = ones;
        ops.push_back(op);
      }
      room -= nops;
    }
    close_batch();
  }
  if ((ops.size() / kBatch) % 2) {  // a batch that copies row 0 to itself
    ops.push_back(Op{0u, 0u, 0u, 0u, one_f, 0u, ones, 0u});
    for (int j = 1; j < kBatch; ++j) ops.push_back(Op{0u, 0u, 0u, ones, 0u, 0u, 0u, 0u});
  }
  table.resize(ops.size() * (sizeof(Op) / 4));
  if (!ops.empty()) __builtin_memcpy(table.data(), ops.data(), ops.size() * sizeof(Op));
  return true;
}

// The table of factor_sequence_kernel from the program above: the program's row operations in order, each put into the
// first group that comes after the writers of the rows it reads and of the row it writes, and not before the readers of
// that row's old value.
void build_factor_entries(const Shape &s, const std::vector<uint32_t> &program, std::vector<uint32_t> &table) {
  struct Terms {
    int dst, cnt;
    uint32_t from[kTerms];
    float w[kTerms];
  };
  const int n = s.n, kGroup = 64 / lanes_per_row(s);
  const uint32_t kRowBytes = 16u * uint32_t(lanes_per_row(s));
  std::vector<Op> ops(program.size() / kOpWords);
  if (!ops.empty()) __builtin_memcpy(ops.data(), program.data(), program.size() * 4);
  std::vector<std::vector<Terms>> groups;
  std::vector<int> written(n, -1), read(n, -1);  // last group that writes or reads a row
  for (size_t k = 0; k < ops.size(); ++k) {
    Terms t{int(ops[k].dst / kProgramRow), 0, {}, {}};
    for (;; ++k) {  // the operations of a row: partial sums to the same row, one after the other
      const Op &op = ops[k];
      float w;
      if (op.m0) __builtin_memcpy(&w, &op.w0, 4), t.from[t.cnt] = op.o0 / kProgramRow, t.w[t.cnt++] = w;
      if (op.m1) __builtin_memcpy(&w, &op.w1, 4), t.from[t.cnt] = op.o1 / kProgramRow, t.w[t.cnt++] = w;
      if ((k + 1) % kBatch == 0 || !ops[k + 1].keep || ops[k + 1].dst != op.dst) break;
    }
    if (t.cnt == 1 && int(t.from[0]) == t.dst && t.w[0] == 1.f) continue;  // a copy of a row to itself fills a batch
    size_t g = size_t(std::max(written[t.dst] + 1, std::max(read[t.dst], 0)));
    for (int i = 0; i < t.cnt; ++i) g = std::max(g, size_t(written[t.from[i]] + 1));
    while (g < groups.size() && int(groups[g].size()) == kGroup) ++g;
    if (g >= groups.size()) groups.resize(g + 1);
    groups[g].push_back(t);
    written[t.dst] = int(g);
    for (int i = 0; i < t.cnt; ++i) read[t.from[i]] = std::max(read[t.from[i]], int(g));
  }
  const uint32_t zero = uint32_t(n) * kRowBytes;
  std::vector<Entry> entries;
  for (const std::vector<Terms> &rows : groups) {
    int slots = 1;
    for (const Terms &t : rows) slots = std::max(slots, (t.cnt + 1) / 2);
    for (int s = 0; s < slots; ++s)
      for (int q = 0; q < kGroup; ++q) {
        const uint32_t to = q < int(rows.size()) ? uint32_t(rows[q].dst) * kRowBytes : zero;
        Entry e{zero | zero << 16, to | (s + 1 == slots ? kLast : 0u), 0.f, 0.f};
        if (q < int(rows.size())) {
          const Terms &t = rows[q];
          if (2 * s < t.cnt) e.from = (e.from & ~0xffffu) | t.from[2 * s] * kRowBytes, e.w0 = t.w[2 * s];
          if (2 * s + 1 < t.cnt) e.from = (e.from & 0xffffu) | t.from[2 * s + 1] * kRowBytes << 16, e.w1 = t.w[2 * s + 1];
        }
        entries.push_back(e);
      }
  }
  while (entries.size() % (kSlotsPadded * kGroup)) entries.push_back(Entry{zero | zero << 16, zero | kLast, 0.f, 0.f});
  table.resize(entries.size() * (sizeof(Entry) / 4));
  if (!entries.empty()) __builtin_memcpy(table.data(), entries.data(), entries.size() * sizeof(Entry));
}

// -1: a tile of n rows does not fit the LDS of a block on this device (the caller applies the factors one by one).
int launch_factor_sequence(const Shape &s, const uint32_t *table, int table_words, void *Z, void *stream) {
  const int lpr = lanes_per_row(s), cols = 4 * lpr, slots = table_words / int(sizeof(Entry) / 4) / (64 / lpr);
  if (slots == 0) return 0;  // every row of every factor is an identity row
  const size_t rows_bytes = size_t(s.n + 1) * 16 * lpr, table_bytes = size_t(table_words) * 4;
  const bool in_lds = table_in_lds(s, rows_bytes, table_bytes);
  const size_t tile_bytes = rows_bytes + (in_lds ? table_bytes : 0), lds_max = size_t(max_lds_per_block());
  // wavefronts per block: whatever keeps most wavefronts on a compute unit, larger blocks on a tie while they
  // stay within the 64 KiB a launch may ask for without raising the kernel's limit
  int waves = 0, resident = 0;
  for (int wv = 1; wv <= 4; wv *= 2) {
    const size_t lds = tile_bytes * wv;
    if (lds > lds_max) break;
    const int res = std::min(int(lds_max / lds) * wv, 32);
    if (res > resident || (res == resident && lds <= 65536)) waves = wv, resident = res;
  }
  if (waves == 0) return -1;
  const size_t lds_bytes = tile_bytes * waves;
  const int64_t piece = kThreadsPerLaunch / 64 * cols;  // columns of one launch
  auto st = static_cast<hipStream_t>(stream);
  auto launch = [&](auto *kernel, auto *z) -> int {
    if (int rc = allow_lds(reinterpret_cast<const void *>(kernel), lds_bytes)) return rc;
    for (int64_t first = 0; first < s.d; first += piece) {
      const int64_t d = std::min(s.d - first, piece);
      kernel<<<dim3(ceil_div_i64(d, int64_t(cols) * waves)), 64 * waves, lds_bytes, st>>>(
          z + first, s.n, d, s.ld, reinterpret_cast<const Entry *>(table), slots);
      if (int rc = hip_rc(hipGetLastError())) return rc;
    }
    return 0;
  };
  auto with = [&](auto lanes, auto access) {
    auto go = [&](auto in_lds) {
      return s.bf16 ? launch(&factor_sequence_kernel<bf16_t, lanes, in_lds, access>, static_cast<bf16_t *>(Z))
                    : launch(&factor_sequence_kernel<float, lanes, in_lds, access>, static_cast<float *>(Z));
    };
    if constexpr (lanes >= 16)
      if (in_lds) return go(std::true_type{});
    return go(std::false_type{});
  };
  auto with_lanes = [&](auto access) {
    return lpr == 32   ? with(std::integral_constant<int, 32>{}, access)
           : lpr == 16 ? with(std::integral_constant<int, 16>{}, access)
                       : with(std::integral_constant<int, 8>{}, access);
  };
  switch (sequence_access(s, Z)) {
    case kStream: return with_lanes(AccessTag<kStream>{});
    case kKeepReads: return with_lanes(AccessTag<kKeepReads>{});
    default: return with_lanes(AccessTag<kKeep>{});
  }
}

}  // namespace detag
