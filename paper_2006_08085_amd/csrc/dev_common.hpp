// Device-side helpers shared by the kernels: state storage types and checks.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace detag {

// bfloat16 storage, handled as raw 16-bit patterns; arithmetic is always fp32.
struct bf16_t {
  uint16_t bits;
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float(uint32_t(v.bits) << 16); }

// Round to nearest, ties to even; NaN stays NaN.  One instruction of gfx950 (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t bf16_bits_rne(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

template <typename ST>
__device__ __forceinline__ ST from_f32(float f);
template <>
__device__ __forceinline__ float from_f32<float>(float f) {
  return f;
}
template <>
__device__ __forceinline__ bf16_t from_f32<bf16_t>(float f) {
  bf16_t r;
  r.bits = bf16_bits_rne(f);
  return r;
}

// Row-tile access through buffer resources.  A resource describes `bytes` valid
// bytes starting at a wavefront-uniform base (tile base + row * pitch); lanes
// address it with a 32-bit byte offset.  The base lives in scalar registers, so
// no per-row 64-bit vector addresses are built, and the hardware range check
// makes out-of-range lanes read zero and drop their stores: ragged tails need
// no branches.
using rsrc_t = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ rsrc_t make_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, int(bytes), 0x00020000);
}

// Row i of a tile: `valid` columns starting at column `tile` of row i.
template <typename E>
__device__ __forceinline__ rsrc_t row_of(const E *base, int64_t tile, int64_t ld, int i, uint32_t valid) {
  return make_rsrc(base + tile + int64_t(i) * ld, valid * uint32_t(sizeof(E)));
}

// How a kernel's accesses treat the caches: kStream marks loads and stores as non-temporal, kKeepReads the stores only,
// kKeep neither.
enum Access : int { kStream, kKeepReads, kKeep };
template <Access A>
using AccessTag = std::integral_constant<Access, A>;

// Cache-policy bits of the buffer instructions on gfx950 (the `aux` operand): bit 0 = sc0, bit 1 = nt, bit 4 = sc1.
template <typename ST, Access A = kStream>
__device__ __forceinline__ float buf_load(rsrc_t r, uint32_t byte_off) {
  constexpr int aux = A == kStream ? 2 : 0;
  if constexpr (sizeof(ST) == 4) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, int(byte_off), 0, aux));
  } else {
    const uint16_t h = uint16_t(__builtin_amdgcn_raw_buffer_load_b16(r, int(byte_off), 0, aux));
    return __uint_as_float(uint32_t(h) << 16);
  }
}

// A value on its way: what a load brings, turned into a float where it is used and not where it was requested.  A kernel that
// keeps the loads of some rows in flight, in an order pinned by scheduling barriers, must not convert next to the load: the
// conversion waits for it (bf16 state, torus 8x8, K = 8, converted at the load and at the use: ATC phase, d = 2,000,000 715 and
// 414 us, 200,000 95 and 54; fused step 705 and 540, with Algorithm 2 as printed 860 and 594; ring of 32, d = 30,000 13.8 and
// 8.0).
template <typename ST>
struct Loaded {
  uint32_t bits;
  __device__ __forceinline__ operator float() const { return __uint_as_float(sizeof(ST) == 4 ? bits : bits << 16); }
};
template <typename ST, Access A = kStream>
__device__ __forceinline__ Loaded<ST> buf_request(rsrc_t r, uint32_t byte_off) {
  constexpr int aux = A == kStream ? 2 : 0;
  if constexpr (sizeof(ST) == 4) return {uint32_t(__builtin_amdgcn_raw_buffer_load_b32(r, int(byte_off), 0, aux))};
  else return {uint32_t(uint16_t(__builtin_amdgcn_raw_buffer_load_b16(r, int(byte_off), 0, aux)))};
}

template <typename ST, Access A = kStream>
__device__ __forceinline__ void buf_store(rsrc_t r, uint32_t byte_off, float v) {
  constexpr int aux = A != kKeep ? 2 : 0;
  if constexpr (sizeof(ST) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, int(byte_off), 0, aux);
  else
    __builtin_amdgcn_raw_buffer_store_b16(short(bf16_bits_rne(v)), r, int(byte_off), 0, aux);
}

// Hides a uniform pointer's value from the optimiser (it stays in scalar
// registers).  Used between the load and the store phase of a tile so the row
// bases are recomputed with a few scalar adds instead of being kept alive, one
// register pair per row, across the whole kernel.
template <typename P>
__device__ __forceinline__ P *launder_uniform(P *p) {
  asm volatile("" : "+s"(p));
  return p;
}

// Forces a value to exist in a vector register at this point of the program.
// Without it the compiler sinks "v = y + gn - go" below the code that does not
// use v yet and carries the three operands instead of the one result.
__device__ __forceinline__ void pin_vgpr(float &v) { asm volatile("" : "+v"(v)); }

// A grid counts its threads in 32 bits, and the runtime launches what is left of a larger number without an error: kernels
// that take many threads per row or column go in pieces of at most this many.
constexpr int64_t kThreadsPerLaunch = int64_t(1) << 31;

inline int hip_rc(hipError_t e) { return static_cast<int>(e); }

inline int ceil_div_i64(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

}  // namespace detag
