// common.hpp -- device-side types and small helpers shared by the HIP kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "hmoe.h"

namespace hmoe {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// Types in LDS (address space 3).  Pointers into shared memory are kept in this address
// space explicitly so that every access compiles to ds_read / ds_write (generic pointers
// would become flat instructions that also wait on outstanding global loads).
template <typename T>
using lds = __attribute__((address_space(3))) T;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16 x) { return (float)x; }

template <typename T>
__device__ __forceinline__ T from_f32(float x);
template <>
__device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <>
__device__ __forceinline__ bf16 from_f32<bf16>(float x) { return (bf16)x; }  // round to nearest even

// Lane-crossing helpers over the 64-wide wavefront.
__device__ __forceinline__ float shfl_xor(float v, int m) { return __shfl_xor(v, m, kWave); }
__device__ __forceinline__ int shfl_xor(int v, int m) { return __shfl_xor(v, m, kWave); }
__device__ __forceinline__ double shfl_xor(double v, int m) { return __shfl_xor(v, m, kWave); }

// v of the lane that a DPP control names, within rows of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// v + v of the lane 32, or 16, away.
template <bool HALVES>
__device__ __forceinline__ float swap_add(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto x = HALVES ? __builtin_amdgcn_permlane32_swap(u, u, false, false)
                        : __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}
template <bool HALVES>
__device__ __forceinline__ double swap_add(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
  const auto lo = HALVES ? __builtin_amdgcn_permlane32_swap(l, l, false, false)
                         : __builtin_amdgcn_permlane16_swap(l, l, false, false);
  const auto hi = HALVES ? __builtin_amdgcn_permlane32_swap(h, h, false, false)
                         : __builtin_amdgcn_permlane16_swap(h, h, false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
// The sum over a row of 16 lanes, in each of them: the rotations by 8, 4, 2, 1 pair the lanes as a
// butterfly does (after a step the values repeat with its distance), so the bits are the same.
template <typename V>
__device__ __forceinline__ V row_sum(V v) {
  v += dpp<0x128>(v);  // row_ror:8, 4, 2, 1
  v += dpp<0x124>(v);
  v += dpp<0x122>(v);
  v += dpp<0x121>(v);
  return v;
}
// The same by distances 1, 2, 4, 8 (a quad's lanes swapped, then halves and rows mirrored).
template <typename V>
__device__ __forceinline__ V row_sum_up(V v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return v;
}
// The butterfly sum over a wave (distances 32 to 1) in registers: six trips through LDS took five
// times as long.  Entered by whole waves.
template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
  return row_sum(swap_add<false>(swap_add<true>(v)));
}

// The four lanes 16 apart (l % 16 alike) combined by `op` without a trip through LDS: two register
// swaps, of odd with even 16-lane rows and of the wave's halves, leave each lane with its own
// and its partner's value.
template <class Op>
__device__ __forceinline__ float rows16_reduce(float v, Op op) {
  typedef unsigned int u2v __attribute__((ext_vector_type(2)));
  const unsigned x = __float_as_uint(v);
  const u2v a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const float p = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const unsigned y = __float_as_uint(p);
  const u2v b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// (value, index) minimum with ties to the lower index.
__device__ __forceinline__ void argmin_merge(float& v, int& i, float v2, int i2) {
  if (v2 < v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

__host__ __device__ __forceinline__ int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Stored decoder logits are offsets from a per-row anchor, one per 64 columns (the row maximum
// over those columns): logit[row][v] = anc[v / 256][row][(v % 256) / 64] + stored[row][v].
constexpr int kAnchorCols = HMOE_ANCHOR_COLS;
constexpr int kAnchorTile = HMOE_ANCHOR_TILE;
constexpr int kAnchorSlots = kAnchorTile / kAnchorCols;
__host__ __device__ __forceinline__ int64_t anchor_index(int64_t n, int64_t row, int64_t col) {
  return ((col / kAnchorTile) * n + row) * kAnchorSlots + (col % kAnchorTile) / kAnchorCols;
}
__host__ __forceinline__ int64_t anchor_count(int64_t n, int64_t vocab) {
  return cdiv(vocab, kAnchorTile) * n * kAnchorSlots;
}

template <typename T>
struct DT;
template <>
struct DT<float> {
  static constexpr hmoe_dtype_t id = HMOE_F32;
};
template <>
struct DT<bf16> {
  static constexpr hmoe_dtype_t id = HMOE_BF16;
};

}  // namespace hmoe
