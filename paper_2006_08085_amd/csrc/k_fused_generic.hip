// The LDS-resident kernels for an arbitrary sparse gossip matrix (layout and round arithmetic in
// fused_generic_common.hpp): plain K-round gossip and the two forms of the DeTAG phase, and the host side that
// packs the neighbour tables.
//
// Paper: Algorithm 3 (accelerated gossip) and Algorithm 2 / the matrix form in
// the proof of Theorem 3 (phase update).
#include <algorithm>
#include <numeric>

#include "fused_generic_common.hpp"

namespace detag {
namespace {

using namespace lds_tile;

// mode 0: Z <- M(Z) on X.  mode 1 (ATC): X <- M(X - alpha*Y), Y <- M(Y + Gn - Go).
// mode 2 (ALG2): X <- M(X) - alpha*M(Y), Y <- M(Y) + Gn - Go.
// mode 3 (D-PSGD): X <- W^T X - alpha*Gn, one plain round (called with eta = 0).
template <typename ST, int MODE, class R, Access A>
__global__ __launch_bounds__(kThreadsMax, R::kWaves) void fused_generic_kernel(ST *X, ST *Y, const float *__restrict__ Gn,
                                                                       const float *__restrict__ Go, int n, int64_t d,
                                                                       int64_t ld, int lpr_log2, typename R::Args ra,
                                                                       float eta, float alpha, int K) {
  Place p{threadIdx.x, blockDim.x, lpr_log2};
  const int64_t first = fused::xcd_tile(blockIdx.x, gridDim.x) << (lpr_log2 + 2);
  const int tile = tile_kind<true, R::kParked != 0>(first, lpr_log2, d);
  f4 z[R::kSlots];
  Waiting<R> v;
  R rounds;  // set up after the first loads: until then its registers are free for them
  auto rows = [&](auto use) { each_row<R, true>(rounds, ra, p, tile, n, d, ld, first, use); };
  auto rows_ahead = [&](auto ahead, auto request, auto use) {
    each_row<ahead, R, true>(rounds, ra, p, tile, n, d, ld, first, request, use);
  };
  constexpr std::integral_constant<int, R::kSlots - 1> kAllAhead;
  // z <- a matrix, all of its loads in flight at once; before(s) comes ahead of those of slot s.
  auto load_all = [&](const ST *from, auto before) {
    if constexpr (std::is_same_v<ST, float>) {
      rows([&](auto F, int s, int64_t off, Columns c, bool) { before(s), z[s] = load4<F, A>(from, off, c, d); });
    } else {
      Raw<ST> r[R::kSlots];
      rows([&](auto F, int s, int64_t off, Columns c, bool) { before(s), r[s] = load4<F, A>(from, off, c, d); });
#pragma unroll
      for (int s = 0; s < R::kSlots; ++s) z[s] = floats(r[s]);
    }
  };
  auto nothing = [](int) {};
  if constexpr (kFetchFirst<R::kSlots>) rounds.fetch(ra, p);
  if constexpr (MODE == 0) {
    load_all(X, nothing);
    rounds.init(ra, p, eta);
    gossip(z, rounds, p, eta, K);
    rows([&](auto F, int s, int64_t off, Columns c, bool mine) { if (mine) store4<F, A>(X, off, c, d, z[s]); });
  } else if constexpr (MODE == 1) {
    // every input is read once: the second gossip's input Y + Gn - Go waits in registers under the first
    struct Row {
      Raw<ST> x, y;
      f4 gn, go;
    };
    auto request = [&](auto F, int, int64_t off, Columns c, int) {
      return Row{load4<F, A>(X, off, c, d), load4<F, A>(Y, off, c, d), load4<F, A>(Gn, off, c, d), load4<F, A>(Go, off, c, d)};
    };
    auto use = [&](auto, int s, int64_t, Columns, bool, const Row &r) {
      const f4 y = floats(r.y);
      z[s] = fma4(-alpha, y, floats(r.x));
      f4 t = y + r.gn - r.go;
      pin4(z[s]), pin4(t);  // the sums now, not their operands carried through the rounds
      v.put(p, s, t);
    };
    constexpr std::integral_constant<int, kAhead<R, 2>> kSomeAhead;
    constexpr std::integral_constant<int, kInOneGo> kNoneAhead;
    // With one weight, fp32 state and few rounds to hide them, blocks of few threads do better with one row's loads at a time,
    // eight neighbours, whose table leaves no register for a row ahead, with any K.  One row at a time and ahead, replayed:
    // 64 workers, 4 neighbours, 3 Mi elements, K = 1 12.8 and 15.6 us, K = 2 14.2 and 15.9, 7 Mi, K = 4 37 and 39, but K = 8
    // 46.3 and 43.7; 24, 4.5 Mi, K = 1 18.6 and 20.6, 12 Mi, K = 8 72 and 66; 128, 4 Mi, K = 1 19 and 20, 200, 12 Mi, K = 2 68
    // and 65, K = 4 79 and 75; 64 workers, 8 neighbours, 4.5 Mi, K = 1 23.0 and 26.9, K = 2 24.9 and 29.8.
    if constexpr (R::kWaves == 8 && std::is_same_v<ST, float>) {
      if (R::kWords > 1 || K * int(blockDim.x) <= 1024) rows_ahead(kNoneAhead, request, use);
      else rows_ahead(kSomeAhead, request, use);
    } else {
      rows_ahead(kSomeAhead, request, use);
    }
    rounds.init(ra, p, eta);
    gossip(z, rounds, p, eta, K);
    rows([&](auto F, int s, int64_t off, Columns c, bool mine) {
      if (mine) store4<F, A>(X, off, c, d, z[s]);
      z[s] = v.get(p, s);
    });
    gossip(z, rounds, p, eta, K);
    rows([&](auto F, int s, int64_t off, Columns c, bool mine) { if (mine) store4<F, A>(Y, off, c, d, z[s]); });
  } else if constexpr (MODE == 3) {
    f4 g[R::kSlots];
    struct Row {
      Raw<ST> x;
      f4 g;
    };
    rows_ahead(kAllAhead, [&](auto F, int, int64_t off, Columns c, int) {
      return Row{load4<F, A>(X, off, c, d), load4<F, A>(Gn, off, c, d)};
    }, [&](auto, int s, int64_t, Columns, bool, const Row &r) {
      z[s] = floats(r.x), g[s] = r.g;
      lds_write(p.own(s), z[s]);
    });
    rounds.init(ra, p, eta);
    __syncthreads();
    rows([&](auto F, int s, int64_t off, Columns c, bool mine) {
      // the increment at its own magnitude and one rounding at that of z, as in the kernel with one launch per round and
      // bit for bit its result (mixed first and -alpha*g added to that: 1.4 to 1.8 times the error against 64 bits); the
      // padded list of a worker without neighbours names itself and is left out
      const f4 mix = n > 1 ? rounds.plain(s, z[s]) : f4{0.f, 0.f, 0.f, 0.f};
      if (mine) store4<F, A>(X, off, c, d, z[s] + fma4(-alpha, g[s], mix));
    });
  } else {
    // M(Y) first: both outputs need it
    load_all(Y, nothing);
    rounds.init(ra, p, eta);
    gossip(z, rounds, p, eta, K);
    load_all(X, [&](int s) { v.put(p, s, z[s]); });
    gossip(z, rounds, p, eta, K);
    // one row's gradients at a time: two rows ahead take eight registers more, and with them a wavefront per SIMD (lists of 64
    // workers, 7 Mi elements, K = 4 48.0 and 42.7 us), a block per compute unit (300 workers, 4 neighbours, 1.8 Mi, K = 4 19.3
    // and 15.5) or spills (200 workers, 8 neighbours, 4.5 Mi, K = 1 29.5 and 24.7)
    rows([&](auto F, int s, int64_t off, Columns c, bool mine) {
      const f4 gn = load4<F, A>(Gn, off, c, d), go = load4<F, A>(Go, off, c, d), my = v.get(p, s);
      if (mine) {
        store4<F, A>(X, off, c, d, fma4(-alpha, my, z[s]));
        store4<F, A>(Y, off, c, d, my + gn - go);
      }
    });
  }
}

template <typename ST, class R>
int launch_r(const Shape &s, const Geometry &g, size_t lds, const typename R::Args &ra, int mode, void *X, void *Y,
             const float *Gn, const float *Go, float alpha, int K, float eta, void *stream) {
  // a lane has 16 elements of a large matrix: 2^36 of them (one bf16 matrix of 137 GB) are 2^32 threads
  const int64_t piece = kThreadsPerLaunch / g.threads * g.cols;  // columns
  auto go = [&](auto *kernel) -> int {
    if (int rc = allow_lds(reinterpret_cast<const void *>(kernel), lds)) return rc;
    for (int64_t first = 0; first < s.d; first += piece) {
      auto at = [&](auto *p) { return p ? p + first : p; };
      const int64_t d = std::min(s.d - first, piece);
      kernel<<<dim3(ceil_div_i64(d, g.cols)), g.threads, lds, static_cast<hipStream_t>(stream)>>>(
          at(static_cast<ST *>(X)), at(static_cast<ST *>(Y)), at(Gn), at(Go), s.n, d, s.ld, g.lpr_log2(), ra, eta, alpha, K);
      if (int rc = hip_rc(hipGetLastError())) return rc;
    }
    return 0;
  };
  auto with = [&](auto access) {
    switch (mode) {
      case 0: return go(&fused_generic_kernel<ST, 0, R, access>);
      case 1: return go(&fused_generic_kernel<ST, 1, R, access>);
      case 2: return go(&fused_generic_kernel<ST, 2, R, access>);
      case 3: return go(&fused_generic_kernel<ST, 3, R, access>);
    }
    return hip_rc(hipErrorInvalidValue);
  };
  const int state = sizeof(ST), per_element = mode == 0 ? state : mode == 3 ? state + 4 : 2 * state + 8;
  const Call call = mode == 0 ? kPlain : mode == 1 ? kAtc : mode == 2 ? kAlg2 : kDpsgd;
  return with_access<R>(s, g, call, per_element, {X, Y, Gn, Go}, with);
}

// Whether a hub makes the kernels with one launch per round the faster ones.  In LDS a wavefront walks the longest list
// alone while the others of its block wait; with three blocks on a compute unit that hides, and up to 32 Mi elements the
// other kernels, whose block walks it too, are slower in any case (star of 257, d = 20,000, K = 8 1390 us against 430).
// Beyond, per round and 1000 columns, fitted to hubs of 64 to 300 neighbours, the other workers on a path or the hub's
// leaves (n = 257 ... 400, d = 150,000, K = 8): 0.12 + 0.0037 longest (two blocks) or 0.22 + 0.0056 longest (one)
// against 0.0022 longest + 0.00073 entries us.  Step of a star of 256 (three blocks) 3320 -> 1990 us, of 257 2970 and
// 3360, of 400 with a hub of 160 on a path 2940 and 2670, of 200 3180 and 3200.
bool lopsided(const Geometry &g, size_t lds, int64_t elements, int longest, int64_t entries) {
  const int blocks = std::min(int(kLdsMax / lds), CsrRounds<kSlotsMax>::kWaves * 4 / (g.threads / 64));
  if (blocks >= 3 || elements <= int64_t(1) << 25) return false;
  return entries < (blocks == 2 ? 2.1 * longest + 164 : 4.6 * longest + 304);
}

}  // namespace

int launch_fused_generic(const Shape &s, const LdsTable &t, int mode, void *X, void *Y, const float *Gn, const float *Go,
                         float alpha, int K, float eta, void *stream) {
  if (K < 1) return -1;
  return with_rounds(s, t, [&](auto r, const Geometry &g, size_t lds, const auto &ra) {
    using R = typename decltype(r)::type;
    return s.bf16 ? launch_r<bf16_t, R>(s, g, lds, ra, mode, X, Y, Gn, Go, alpha, K, eta, stream)
                  : launch_r<float, R>(s, g, lds, ra, mode, X, Y, Gn, Go, alpha, K, eta, stream);
  });
}

bool build_lds_table(const HostW &W, int64_t d, LdsTableHost &out) {
  const int n = W.n;
  int maxdeg = 0;
  int64_t entries = 0;  // off the diagonal
  bool one_weight = true, have = false;
  float weight = 0.f;
  for (int i = 0; i < n; ++i) {
    int cnt = 0;
    for (int k = W.rowptr[i]; k < W.rowptr[i + 1]; ++k) {
      if (W.colidx[k] == i) continue;
      const float v = float(W.vals[k]);
      if (!have) weight = v, have = true;
      else if (v != weight) one_weight = false;
      ++cnt;
    }
    maxdeg = std::max(maxdeg, cnt), entries += cnt;
  }
  out = LdsTableHost{};
  // a small matrix of more workers than two rows per lane of a 64-column tile hold (n > 128) is better off with the
  // lists, whose tiles go down to 16 columns: n = 200, d = 4,000, K = 12 16 against 33 us
  const bool byte_form = n <= kByteRows && maxdeg <= 8 && one_weight &&
                         (!small_matrix(n, d) || byte_geometry(n, d).slots < kSlotsMax);
  if (byte_form) {
    out.bytes_deg = maxdeg <= 2 ? 2 : maxdeg <= 4 ? 4 : 8;
    out.weight = weight;
    const int words = out.bytes_deg <= 4 ? 1 : 2;
    out.byte_table.assign(size_t(kByteRows) * words, 0u);
    for (int i = 0; i < kByteRows; ++i) {
      uint8_t nb[8];
      for (uint8_t &b : nb) b = uint8_t(i);  // a missing neighbour is the row itself: difference zero
      int cnt = 0;
      if (i < n)
        for (int k = W.rowptr[i]; k < W.rowptr[i + 1]; ++k)
          if (W.colidx[k] != i) nb[cnt++] = uint8_t(W.colidx[k]);
      for (int k = 0; k < 4 * words; ++k) out.byte_table[size_t(i) * words + k / 4] |= uint32_t(nb[k]) << (8 * (k % 4));
    }
    return true;
  }
  const Geometry g = csr_geometry(n, d);
  if (g.cols == 0) return false;
  const int positions = g.positions(), lpr = g.cols / 4, rows_per_wave = 64 / lpr, waves = g.threads / 64;
  const int per_slot = g.threads / lpr;
  auto offset = [&](int p) { return uint32_t(p) * g.cols * 4u; };
  // with weights of their own the lists stay in LDS: offsets in registers (16 of them, and one wavefront less per SIMD) and
  // only the weights there measured -16 to +13 % (D-PSGD step and Algorithm 2's phase of 48 and 200 irregular workers 112 ->
  // 125 us and 153 -> 166)
  if (g.slots == kSlotsMax && maxdeg <= 8 && one_weight) {
    out.half_deg = maxdeg <= 2 ? 2 : maxdeg <= 4 ? 4 : 8;
    out.weight = weight;
    out.offsets.assign(size_t(positions) * out.half_deg / 2, 0u);
    for (int i = 0; i < positions; ++i) {  // a row sits at its own number
      size_t k = size_t(i) * out.half_deg;
      auto put = [&](uint32_t off) { out.offsets[k / 2] |= off << (16 * (k % 2)), ++k; };
      if (i < n)
        for (int t = W.rowptr[i]; t < W.rowptr[i + 1]; ++t)
          if (W.colidx[t] != i) put(offset(W.colidx[t]));
      while (k < size_t(i + 1) * out.half_deg) put(offset(i));  // a missing neighbour is the row itself: difference zero
    }
    return true;
  }
  // rows by falling degree; slot by slot, every other slot from the last wavefront to the first, so that no wavefront
  // gets the longest lists of every slot
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  auto degree = [&](int i) { return W.rowptr[i + 1] - W.rowptr[i]; };
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return degree(a) > degree(b); });
  out.rows.assign(positions, -1);
  std::vector<int> position(n);
  int next = 0;
  for (int s = 0; s < g.slots && next < n; ++s)
    for (int q = 0; q < waves && next < n; ++q) {
      const int w = s % 2 ? waves - 1 - q : q;
      for (int k = 0; k < rows_per_wave && next < n; ++k) {
        const int p = s * per_slot + w * rows_per_wave + k;
        out.rows[p] = order[next], position[order[next]] = p, ++next;
      }
    }
  for (int w = 0; w < waves; ++w)
    for (int s = 0; s < g.slots; ++s) {
      const int p0 = s * per_slot + w * rows_per_wave;
      std::vector<std::vector<std::pair<uint32_t, float>>> lists(rows_per_wave);
      size_t pairs = 0;
      for (int k = 0; k < rows_per_wave; ++k) {
        const int i = out.rows[p0 + k];
        if (i >= 0)
          for (int t = W.rowptr[i]; t < W.rowptr[i + 1]; ++t)
            if (W.colidx[t] != i) lists[k].push_back({offset(position[W.colidx[t]]), float(W.vals[t])});
        pairs = std::max(pairs, (lists[k].size() + 1) / 2);
      }
      out.groups.push_back(uint32_t(out.pairs.size() / 4)), out.groups.push_back(uint32_t(pairs));
      out.max_pairs = std::max(out.max_pairs, int(pairs));
      for (size_t q = 0; q < pairs; ++q)
        for (int k = 0; k < rows_per_wave; ++k)
          for (size_t e = 2 * q; e < 2 * q + 2; ++e) {
            const bool there = e < lists[k].size();
            out.pairs.push_back(there ? lists[k][e].first : offset(p0 + k));  // or the row itself, weight 0
            const float v = there ? lists[k][e].second : 0.f;
            uint32_t bits;
            __builtin_memcpy(&bits, &v, sizeof bits);
            out.pairs.push_back(bits);
          }
    }
  const size_t lds = g.tile_bytes(0) + out.pairs.size() * 4;
  if (lds > kLdsMax || lopsided(g, lds, n * d, maxdeg, entries)) {
    out = LdsTableHost{};
    return false;
  }
  return true;
}

}  // namespace detag
