// Gradient query of the diagonal-quadratic objective fused into the ATC phase of the LDS-resident kernels
// (layout and round arithmetic in fused_generic_common.hpp).
//
// Paper: gradient query and phase update of Algorithm 2 (matrix form in the proof of Theorem 3), Algorithm 3.
#include "fused_generic_common.hpp"
#include "noise_dev.hpp"

namespace detag {
namespace {

using namespace lds_tile;

// Gradient query of the diagonal-quadratic objective and the ATC phase in one pass (the form
// detag_step_quadratic takes on a context of this kernel family):
//   G+ = h*(X - b) + sigma*z;  X+ = M(X - alpha*Y);  Y+ = M(Y + G+ - G),
// G updated in place (row by row, the old value read just before the new one is stored).  Same three arrays
// per lane as the plain ATC phase: the gradient is consumed and stored inside the load loop.  Per element it
// reads X, Y (state type), G, b (fp32) and writes X, Y, G, where the gradient kernel followed by the phase moves
// X twice more and the gradient three times.  A lane's four columns of a row are one Philox block of the
// counter-based noise.
template <typename ST, bool HPW, class R, Access A>
__global__ __launch_bounds__(kThreadsMax, R::kWaves) void fused_generic_quadratic_kernel(
    ST *X, ST *Y, float *G, const float *__restrict__ h, const float *__restrict__ b, int n, int64_t d, int64_t ld,
    int lpr_log2, typename R::Args ra, float eta, float alpha, int K, float sigma, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t step) {
  Place p{threadIdx.x, blockDim.x, lpr_log2};
  const int64_t first = fused::xcd_tile(blockIdx.x, gridDim.x) << (lpr_log2 + 2);
  // within 64 registers the third form of the loads costs the others a spill (n = 256, d = 1 M, bf16, K = 4 1167 -> 1189 us)
  constexpr bool kCutTiles = R::kParked == 0;
  const int tile = tile_kind<kCutTiles, R::kParked != 0>(first, lpr_log2, d);
  f4 z[R::kSlots];
  Waiting<R> v;
  R rounds;  // set up after the loads: until then its registers are free for them
  auto rows = [&](auto use) { each_row<R, kCutTiles>(rounds, ra, p, tile, n, d, ld, first, use); };
  if constexpr (kFetchFirst<R::kSlots>) rounds.fetch(ra, p);
  struct Row {
    f4 noise, b, h, go;
    Raw<ST> x, y;
  };
  each_row<kAhead<R, 1>, R, kCutTiles>(rounds, ra, p, tile, n, d, ld, first, [&](auto F, int, int64_t off, Columns c, int row) {
    // the row's noise first, its loads after: generated under the loads, the Philox state and the values in flight
    // are live together and the kernel does not fit its registers
    Row r;
    r.noise = f4{0.f, 0.f, 0.f, 0.f};
    if (sigma != 0.f) {
      float t[4];
      normal4(uint64_t(c.at + c.skip) >> 2, uint32_t(row), step, seed_lo, seed_hi, t);
      r.noise = f4{t[0], t[1], t[2], t[3]};
      if (F == kCut && c.skip > 0)  // the block of the lane's own columns, moved to where they are
        r.noise = f4{t[0], c.skip == 1 ? t[0] : t[1], c.skip == 1 ? t[1] : t[0], c.skip == 1 ? t[2] : c.skip == 2 ? t[1] : t[0]};
    }
    __builtin_amdgcn_sched_barrier(0);
    r.x = load4<F, A>(X, off, c, d), r.b = load4<F, A>(b, off, c, d), r.h = load4<F, A>(h, HPW ? off : 0, c, d);
    r.y = load4<F, A>(Y, off, c, d), r.go = load4<F, A>(G, off, c, d);
    return r;
  }, [&](auto F, int s, int64_t off, Columns c, bool mine, const Row &r) {
    f4 g;
    const f4 x = floats(r.x), y = floats(r.y);
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = fmaf(sigma, r.noise[e], r.h[e] * (x[e] - r.b[e]));
    z[s] = fma4(-alpha, y, x);
    f4 t = y + g - r.go;
    pin4(z[s]), pin4(t);
    v.put(p, s, t);
    if (mine) store4<F, A>(G, off, c, d, g);
  });
  rounds.init(ra, p, eta);
  gossip(z, rounds, p, eta, K);
  rows([&](auto F, int s, int64_t off, Columns c, bool mine) {
    if (mine) store4<F, A>(X, off, c, d, z[s]);
    z[s] = v.get(p, s);
  });
  gossip(z, rounds, p, eta, K);
  rows([&](auto F, int s, int64_t off, Columns c, bool mine) { if (mine) store4<F, A>(Y, off, c, d, z[s]); });
}

}  // namespace

int launch_fused_generic_quadratic(const Shape &s, const LdsTable &t, void *X, void *Y, float *G, const float *h,
                                   bool h_per_worker, const float *b, float alpha, int K, float eta, float sigma,
                                   uint64_t seed, uint32_t step, void *stream) {
  if (K < 1) return -1;
  return with_rounds(s, t, [&](auto r, const Geometry &g, size_t lds, const auto &ra) {
    using R = typename decltype(r)::type;
    if constexpr (std::is_same_v<typename R::Args, HalfArgs>) {
      return -1;  // more than 256 workers: no fused step
    } else {
      auto go = [&](auto *kernel, auto *x, auto *y) -> int {
        if (int rc = allow_lds(reinterpret_cast<const void *>(kernel), lds)) return rc;
        kernel<<<dim3(ceil_div_i64(s.d, g.cols)), g.threads, lds, static_cast<hipStream_t>(stream)>>>(
            x, y, G, h, b, s.n, s.d, s.ld, g.lpr_log2(), ra, eta, alpha, K, sigma, uint32_t(seed & 0xffffffffu),
            uint32_t(seed >> 32), step);
        return hip_rc(hipGetLastError());
      };
      auto with = [&](auto access) {
        if (s.bf16) {
          auto *x = static_cast<bf16_t *>(X), *y = static_cast<bf16_t *>(Y);
          return h_per_worker ? go(&fused_generic_quadratic_kernel<bf16_t, true, R, access>, x, y)
                              : go(&fused_generic_quadratic_kernel<bf16_t, false, R, access>, x, y);
        }
        auto *x = static_cast<float *>(X), *y = static_cast<float *>(Y);
        return h_per_worker ? go(&fused_generic_quadratic_kernel<float, true, R, access>, x, y)
                            : go(&fused_generic_quadratic_kernel<float, false, R, access>, x, y);
      };
      const int per_element = (s.bf16 ? 4 : 8) + 8 + (h_per_worker ? 4 : 0);
      // blocks of 1024 threads, two to a compute unit, are better off streaming: 256 x 30,001 53.3, 62.8, 72.2 us
      const Call call = g.threads <= 512 ? kFusedStep : kAtc;
      return with_access<R>(s, g, call, per_element, {X, Y, G, h_per_worker ? h : nullptr, b}, with);
    }
  });
}

}  // namespace detag
