// Mini-batch gradient of multinomial logistic regression, every worker on its
// own batch (the gradient query of Algorithm 2 for the label-sorted-shard
// workload), in two launches (three from 6,145 features on):
//
//   logits[s,c] = sum_f feat[s,f] * Wt[c,f] + bias[c]        (B x F) . (F x C)
//   dW[c,f]     = sum_s delta[s,c] * feat[s,f]                (C x B) . (B x F)
//
// The features are bf16 data, weights and residuals fp32.  The batch of 32 workers x 128 samples x 3072 features is 25 MB,
// read by both launches (the second time mostly from the memory-side cache): what bounds them is how many of those bytes
// are in flight and how long the chain index - row - sum - softmax is, not arithmetic.  So both launches cut the features
// into up to 16 blocks per worker, one per compute unit from 16 workers with wide features on, and a wavefront requests
// all the feature bytes it needs before it uses the first.
//
//   softmax_logits_kernel  block = one worker x one chunk of up to 384 features x the whole batch, one wavefront per 16
//     samples.  The products run on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate); the chunk's
//     weights are split exactly into three bf16 terms w = hi + mid + lo on the way into LDS, once per block, so the
//     products carry every bit of the fp32 weights.  Writes the chunk's part of the logits.
//   softmax_grad_kernel    the same blocks, a wavefront per 32 features.  Workgroups go to the eight XCDs in turn, so a
//     block finds in its XCD's L2 what the same block of the first launch read (25 MB spread over 8 x 4 MB).  Every
//     block adds up the parts of the logits and takes the softmax itself (10 x 128 values, while its feature rows
//     arrive): a launch in between, or a ticket for the last block, costs more.  The residuals are split into three
//     bf16 terms in LDS; a wavefront transposes its features through an LDS area of its own, 64 samples at a time, and
//     multiplies on the matrix cores.  (The products in fp32 on the vector ALUs, samples shared among the wavefronts
//     and summed in LDS at the end, took 16 to 17 us: 4.9 us of multiplications and a 3 us tail.)
// The times at the two kernels are for 32 workers, 128 samples, 3072 features and 10 classes; with the phase after them
// the call takes 25.8 us.
//
// MFMA 16x16x32 operand layout (lane l, m = l % 16, q = l / 16):
//   A: row m, k = 8q..8q+7      B: column m, k = 8q..8q+7
//   D: column m, register r -> row 4q + r
#include <algorithm>

#include "dev_common.hpp"
#include "detag_internal.h"

namespace detag {
namespace {

constexpr int kClassesMax = 10, kSamplesMax = 256;
constexpr int kChunkMax = 384, kStepsMax = kChunkMax / 32;  // features of a logits block, MFMA steps of 32
constexpr int kWeightPitch = kChunkMax + 8;  // bf16 per weight row in LDS: 16 rows start in 16 different groups of 4 banks
constexpr int kGradWaves = kChunkMax / 32, kGradThreads = 64 * kGradWaves;
constexpr int kWaveCols = 32;     // features of a wavefront
constexpr int kStage = 64;        // samples a wavefront transposes at a time
constexpr int kStagePitch = 36;   // bf16 per staged row, 72 B: rows 8 apart start 64 B apart in the banks
constexpr int kHeld = 2;          // stages whose rows are requested together
constexpr int kDeltaPitch = kSamplesMax + 8;  // bf16 per class and term: 16 classes start in 16 groups of 4 banks
constexpr int kLanesClasses = 12;  // classes four lanes of a sample cover

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// The exact three-way split w = hi + mid + lo, each a bf16.
__device__ __forceinline__ void bf16_split(float w, uint16_t (&t)[3]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    t[p] = bf16_bits_rne(w);
    w -= __uint_as_float(uint32_t(t[p]) << 16);
  }
}

__device__ __forceinline__ int clamped(int v, int n) { return v < 0 ? 0 : v >= n ? n - 1 : v; }

// grid (chunks, n), B/16 wavefronts.  part[i][chunk][c][s] = sum over the chunk's features.
// 32 workers x 8 chunks: 7.4 us (formerly a splitting kernel, 5.7 us, and 128 blocks that split the features over 16
// wavefronts and summed in LDS, 20.7 us).
__global__ __launch_bounds__(64 * kSamplesMax / 16) void softmax_logits_kernel(
    int64_t ld, const float *__restrict__ X, const uint16_t *__restrict__ feat, const int32_t *__restrict__ batch, int S, int F,
    int C, int B, int chunk, float *__restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint16_t weight[3][kClassesMax][kWeightPitch];
  const int i = blockIdx.y, f0 = blockIdx.x * chunk, nf = F - f0 < chunk ? F - f0 : chunk, steps = nf / 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int idx = clamped(batch[int64_t(i) * B + wave * 16 + m], S);
  const uint16_t *frow = feat + (int64_t(i) * S + idx) * F + f0 + 8 * q;
  // the weights are asked for ahead of the features, which wait for the numbers of the samples, and split while those arrive
  // (behind them 32 workers, 128 samples, 3072 features 8.6 us, so 7.4; 8, 32 samples, 64 features 3.8 and 3.1;
  // but 32, 256 samples, 4096 features 17.4 and 18.0)
  auto weights = [&](int k) {
    const int c = k / nf, f = k % nf;  // nf is a multiple of 32: the four stay in a row
    return *reinterpret_cast<const f32x4_any *>(X + int64_t(i) * ld + int64_t(c) * F + f0 + f);
  };
  constexpr int kFirst = 2;
  const int step = blockDim.x * 4;
  f32x4 first[kFirst];
#pragma unroll
  for (int j = 0; j < kFirst; ++j) {
    const int k = threadIdx.x * 4 + j * step;
    if (j * step < C * nf) first[j] = weights(k < C * nf ? k : 0);  // uniform
  }
  __builtin_amdgcn_sched_barrier(0);
  u16x8 fv[kStepsMax];
#pragma unroll
  for (int st = 0; st < kStepsMax; ++st)
    if (st < steps) fv[st] = *reinterpret_cast<const u16x8 *>(frow + 32 * st);  // uniform condition
  __builtin_amdgcn_sched_barrier(0);
  auto split = [&](int k, f32x4 w) {
    const int c = k / nf, f = k % nf;
    u16x4 t[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint16_t s[3];
      bf16_split(w[e], s);
      t[0][e] = s[0], t[1][e] = s[1], t[2][e] = s[2];
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<u16x4 *>(&weight[p][c][f]) = t[p];
  };
#pragma unroll
  for (int j = 0; j < kFirst; ++j) {
    const int k = threadIdx.x * 4 + j * step;
    if (k < C * nf) split(k, first[j]);
  }
  for (int k = threadIdx.x * 4 + kFirst * step; k < C * nf; k += step) split(k, weights(k));
  __syncthreads();
  const int row = m < C ? m : C - 1;  // rows past C of the tile repeat the last class and are not stored
  // the upper term and the two small ones in accumulators of their own: added to one, the small terms would triple the
  // roundings at the magnitude of the sum
  f32x4 acc = {0.f, 0.f, 0.f, 0.f}, low = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < kStepsMax; ++st)
    if (st < steps) {
      auto product = [&](int p, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&weight[p][row][32 * st + 8 * q])),
            __builtin_bit_cast(bf16x8, fv[st]), c, 0, 0, 0);
      };
      low = product(2, low);
      acc = product(0, acc);
      low = product(1, low);
    }
  acc += low;
  float *out = part + (int64_t(i) * gridDim.x + blockIdx.x) * C * B + wave * 16 + m;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (4 * q + r < C) out[int64_t(4 * q + r) * B] = acc[r];
}

// grid (chunks, n).  32 workers x 8 chunks: 11.8 us; with column groups that do not match the first launch's, whose
// features then come from beyond the L2, 15.6 us then.
__global__ __launch_bounds__(kGradThreads) void softmax_grad_kernel(
    int64_t ld, const float *__restrict__ X, const uint16_t *__restrict__ feat, const int32_t *__restrict__ labels,
    const int32_t *__restrict__ batch, int S, int F, int C, int B, int chunk, const float *__restrict__ part, int parts,
    float *__restrict__ G, float *__restrict__ loss) {
  __shared__ __attribute__((aligned(16))) uint16_t delta[3][kClassesMax][kDeltaPitch];
  __shared__ __attribute__((aligned(16))) uint16_t stages[kGradWaves][kStage][kStagePitch];
  __shared__ float logits[kClassesMax * kSamplesMax], sample_loss[kSamplesMax];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int i = blockIdx.y, f0 = blockIdx.x * chunk + wave * kWaveCols;
  part += int64_t(i) * gridDim.x * C * B;
  const bool cols_ok = wave * kWaveCols < chunk && f0 < F;  // F % 32 == 0: a wavefront's columns are all in or all out
  const int32_t *rows = batch + int64_t(i) * B;
  // a stage's rows: four lanes to a row of 64 B, sixteen rows an instruction
  u16x8 v[kHeld][kStage / 16];
  int at[kHeld][kStage / 16];
  auto each_piece = [&](int from, auto f) {
#pragma unroll
    for (int h = 0; h < kHeld; ++h)
#pragma unroll
      for (int k = 0; k < kStage / 16; ++k) {
        const int s = from + h * kStage + k * 16;  // uniform; B is a multiple of 32
        if (cols_ok && s < B) f(h, k, s);
      }
  };
  auto find = [&](int from) { each_piece(from, [&](int h, int k, int s) { at[h][k] = rows[s + (lane >> 2)]; }); };
  auto fetch = [&](int from) {
    each_piece(from, [&](int h, int k, int) {
      v[h][k] = *reinterpret_cast<const u16x8 *>(feat + (int64_t(i) * S + clamped(at[h][k], S)) * F + f0 + (lane & 3) * 8);
    });
  };
  // Memory answers a wavefront in the order it asked: the numbers of the samples first, on which labels and features wait,
  // then the parts of the logits and the bias, the labels, and the feature rows, which arrive under the softmax.  (Numbers
  // behind the parts and the bias behind the features, each a latency more in the chain: 32 workers, 256 samples, 4096
  // features 33.1 us, so 26.4; 4, 160 samples, 1024 features 10.4 and 8.7; 32, 128 samples, 3072 features 12.6 and 11.8.)
  // This thread's (class, sample) pairs:
  constexpr int kPairs = (kClassesMax * kSamplesMax + kGradThreads - 1) / kGradThreads;
  constexpr int kPasses = (kSamplesMax * 4 + kGradThreads - 1) / kGradThreads;
  float sums[kPairs];
  // four lanes share a sample: lane j takes classes j, j + 4, j + 8
  int y[kPasses];
  float bias[kPairs];
#pragma unroll
  for (int r = 0; r < kPasses; ++r) {
    const int s = int(threadIdx.x) / 4 + r * (kGradThreads / 4);
    y[r] = rows[s < B ? s : 0];
  }
  find(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < kPairs; ++j) {
    const int k = int(threadIdx.x) + j * kGradThreads;
    sums[j] = 0.f;
    bias[j] = k < C * B ? X[int64_t(i) * ld + int64_t(C) * F + k / B] : 0.f;
  }
  for (int q0 = 0; q0 < parts; q0 += 8) {
    float t[kPairs][8];
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
      const int k = int(threadIdx.x) + j * kGradThreads;
      if (j * kGradThreads < C * B) {  // uniform
#pragma unroll
        for (int q = 0; q < 8; ++q)
          t[j][q] = k < C * B && q0 + q < parts ? part[int64_t(q0 + q) * C * B + k] : 0.f;
      }
    }
    if (q0 + 8 >= parts) {
#pragma unroll
      for (int r = 0; r < kPasses; ++r) {
        const int s = int(threadIdx.x) / 4 + r * (kGradThreads / 4);
        y[r] = s < B ? labels[int64_t(i) * S + clamped(y[r], S)] : 0;
      }
      fetch(0);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < kPairs; ++j)
      if (j * kGradThreads < C * B) {
#pragma unroll
        for (int q = 0; q < 8; ++q) sums[j] += t[j][q];
      }
  }
#pragma unroll
  for (int j = 0; j < kPairs; ++j) {
    const int k = int(threadIdx.x) + j * kGradThreads;
    if (k < C * B) {
      const int c = k / B;
      logits[c * kSamplesMax + k % B] = sums[j] + bias[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPasses; ++r) {
    const int s = int(threadIdx.x) / 4 + r * (kGradThreads / 4), j = threadIdx.x & 3;
    y[r] = clamped(y[r], C);
    if (s < B) {  // the four lanes of a sample together
      float e[kLanesClasses / 4], mx = -__builtin_inff();
#pragma unroll
      for (int k = 0; k < kLanesClasses / 4; ++k) {
        const int c = j + 4 * k;
        e[k] = c < C ? logits[c * kSamplesMax + s] : -__builtin_inff();
        mx = fmaxf(mx, e[k]);
      }
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
      float sum = 0.f, of_y = 0.f;
#pragma unroll
      for (int k = 0; k < kLanesClasses / 4; ++k) {
        e[k] = j + 4 * k < C ? expf(e[k] - mx) : 0.f;
        sum += e[k];
        if (j + 4 * k == y[r]) of_y = e[k];
      }
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) sum += __shfl_xor(sum, o, 64), of_y += __shfl_xor(of_y, o, 64);
      const float inv = 1.f / sum, invB = 1.f / float(B);
#pragma unroll
      for (int k = 0; k < kLanesClasses / 4; ++k) {
        const int c = j + 4 * k;
        if (c < C) {
          const float dl = (e[k] * inv - (c == y[r] ? 1.f : 0.f)) * invB;
          uint16_t t[3];
          bf16_split(dl, t);
#pragma unroll
          for (int p = 0; p < 3; ++p) delta[p][c][s] = t[p];
          logits[c * kSamplesMax + s] = dl;  // for the bias gradient; only these four lanes read the sample's logits
        }
      }
      if (j == 0) sample_loss[s] = -logf(of_y * inv);
    }
  }
  __syncthreads();
  if (cols_ok) {
    f32x4 acc[2], low[2];
    acc[0] = acc[1] = low[0] = low[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int row = m < C ? m : C - 1;  // rows past C of the tile repeat the last class and are not stored
    uint16_t(&stage)[kStage][kStagePitch] = stages[wave];
    for (int from = 0; from < B; from += kHeld * kStage) {
      if (from > 0) find(from), fetch(from);
#pragma unroll
      for (int h = 0; h < kHeld; ++h) {
        const int s0 = from + h * kStage;
        if (s0 >= B) break;
        // LDS serves a wavefront in order: the rows are written before they are read, and read before the next stage's
#pragma unroll
        for (int k = 0; k < kStage / 16; ++k)
          if (s0 + k * 16 < B) {
            u16x4 *to = reinterpret_cast<u16x4 *>(&stage[k * 16 + (lane >> 2)][(lane & 3) * 8]);
            to[0] = u16x4{v[h][k][0], v[h][k][1], v[h][k][2], v[h][k][3]};
            to[1] = u16x4{v[h][k][4], v[h][k][5], v[h][k][6], v[h][k][7]};
          }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int st = 0; st < kStage / 32; ++st)
          if (s0 + st * 32 < B) {
            u16x8 a[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) a[p] = *reinterpret_cast<const u16x8 *>(&delta[p][row][s0 + st * 32 + 8 * q]);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              u16x8 x;
#pragma unroll
              for (int j = 0; j < 8; ++j) x[j] = stage[st * 32 + 8 * q + j][t * 16 + m];
              auto product = [&](int p, f32x4 c) {
                return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[p]), __builtin_bit_cast(bf16x8, x), c,
                                                               0, 0, 0);
              };
              low[t] = product(2, low[t]);
              acc[t] = product(0, acc[t]);
              low[t] = product(1, low[t]);
            }
          }
        __builtin_amdgcn_wave_barrier();
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * q + r < C) G[int64_t(i) * ld + int64_t(4 * q + r) * F + f0 + t * 16 + m] = acc[t][r] + low[t][r];
  }
  if (blockIdx.x == 0) {
    // bias gradient: sum over the batch of delta (already divided by B); wavefront w takes classes w, w+8
    for (int c = wave; c < C; c += kGradWaves) {
      float sum = 0.f;
      for (int s = threadIdx.x & 63; s < B; s += 64) sum += logits[c * kSamplesMax + s];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o, 64);
      if ((threadIdx.x & 63) == 0) G[int64_t(i) * ld + int64_t(C) * F + c] = sum;
    }
    if (wave == kGradWaves - 1 && loss) {
      float sum = 0.f;
      for (int s = threadIdx.x & 63; s < B; s += 64) sum += sample_loss[s];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o, 64);
      if ((threadIdx.x & 63) == 0) loss[i] = sum / float(B);
    }
  }
}

// Adds up the parts of the logits where there are many, into the place of the first.  grid (C*B / 64, n): a wavefront takes
// every sixteenth part of 64 values.
constexpr int kSumWaves = 16;
__global__ __launch_bounds__(64 * kSumWaves) void softmax_sum_kernel(int values, int parts, float *__restrict__ part) {
  __shared__ float sums[kSumWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, k = blockIdx.x * 64 + lane;
  float *mine = part + int64_t(blockIdx.y) * parts * values + k;
  float sum = 0.f;
  if (k < values) {
#pragma unroll 8
    for (int q = wave; q < parts; q += kSumWaves) sum += mine[int64_t(q) * values];
  }
  sums[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && k < values) {
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < kSumWaves; ++w) sum += sums[w][lane];
    *mine = sum;
  }
}

// Features per logits block: enough chunks that n workers make 256 blocks, at most 16 (every gradient block adds the
// parts up), a multiple of 32.
int logits_chunk(int n, int F) {
  const int64_t chunks = std::min((256 + n - 1) / n, 16), chunk = ((F + chunks - 1) / chunks + 31) / 32 * 32;
  return int(std::min<int64_t>(chunk, kChunkMax));
}
int logits_chunks(int n, int F) { return ceil_div_i64(F, logits_chunk(n, F)); }

// With more parts than this a launch adds them up once.  Every gradient block would otherwise read them all, which grows
// with the square of the features: 32 workers, 128 samples, 10 classes, 150,528 features 3220 us without it, 830 with it;
// 8,192 features (22 parts) 52 and 48 us.  At 16 parts and below the launch costs what it saves (6,144 features 36.5 and
// 36.4 us; 8 workers, 64 samples 15.0 and 16.1 us).
constexpr int kPartsMax = 16;

}  // namespace

// The parts of the logits, n x chunks x C x B.
int64_t softmax_scratch_floats(int n, int C, int B, int F) { return int64_t(n) * logits_chunks(n, F) * C * B; }

int launch_grad_softmax(const Shape &s, const void *X, const uint16_t *feat, const int32_t *labels,
                        const int32_t *batch, int S, int F, int C, int B, float *scratch, float *G, float *loss,
                        void *stream) {
  auto st = static_cast<hipStream_t>(stream);
  const float *x = static_cast<const float *>(X);
  const int chunk = logits_chunk(s.n, F), chunks = logits_chunks(s.n, F);
  softmax_logits_kernel<<<dim3(chunks, s.n), 64 * (B / 16), 0, st>>>(s.ld, x, feat, batch, S, F, C, B, chunk, scratch);
  if (int rc = hip_rc(hipGetLastError())) return rc;
  if (chunks > kPartsMax) {
    softmax_sum_kernel<<<dim3((C * B + 63) / 64, s.n), 64 * kSumWaves, 0, st>>>(C * B, chunks, scratch);
    if (int rc = hip_rc(hipGetLastError())) return rc;
  }
  softmax_grad_kernel<<<dim3(chunks, s.n), kGradThreads, 0, st>>>(s.ld, x, feat, labels, batch, S, F, C, B, chunk, scratch,
                                                                  chunks > kPartsMax ? 1 : chunks, G, loss);
  return hip_rc(hipGetLastError());
}

}  // namespace detag
