// storage.hpp -- encodings of the stored population deviations (FP32, FP16, BF16)
// and the AA-pattern slot of population i at node x.
//
// The stored value is q = (f_i - w_i rho0) / sigma_class(i); sigma is 1 for FP32
// and the thermal scale sqrt(w_i rho0 kT / cs^2) (or a user scale) for 16-bit
// storage, so thermal noise is O(1) in storage units.  Stores round to nearest
// even.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace rflbm {

template <int S>
struct Codec;

// decode(q, sigma) = q sigma; decode_add(q, sigma, c) = q sigma + c and
// decode_sub(q, sigma, c) = c - q sigma, each one rounding (a fused
// multiply-add, or an exact add where sigma is 1).  SPLIT (FP16): widen and
// multiply-add by two instructions, which issue faster than the one
// mixed-precision instruction the compiler takes otherwise; the same value.  The
// one-box steps use it (64^3 9.09 -> 8.50 us, 128^3 43.0 -> 40.8, 512^3 2717 ->
// 2692), not those with a box offset per lane (96^3 20.1 -> 21.1).  The store stays
// one instruction: a product and a conversion round twice, which changes the
// totals that 16-bit rounding moves.
template <>
struct Codec<kF32> {
  using T = float;
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode(T q, float) { return q; }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_add(T q, float, float c) { return q + c; }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_sub(T q, float, float c) { return c - q; }
  __device__ __forceinline__ static T encode(float d, float) { return d; }
};

template <>
struct Codec<kF16> {
  using T = _Float16;
  template <bool SPLIT>
  __device__ __forceinline__ static float widen(T q) {
    float x = static_cast<float>(q);
    if constexpr (SPLIT) asm volatile("" : "+v"(x));
    return x;
  }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode(T q, float sigma) { return widen<SPLIT>(q) * sigma; }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_add(T q, float sigma, float c) {
    return fmaf(widen<SPLIT>(q), sigma, c);
  }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_sub(T q, float sigma, float c) {
    return fmaf(widen<SPLIT>(q), -sigma, c);
  }
  __device__ __forceinline__ static T encode(float d, float inv_sigma) {
    return static_cast<_Float16>(d * inv_sigma);
  }
};

template <>
struct Codec<kBF16> {
  using T = uint16_t;  // raw bfloat16 bits
  __device__ __forceinline__ static float widen(T q) { return __uint_as_float(static_cast<uint32_t>(q) << 16); }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode(T q, float sigma) { return widen(q) * sigma; }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_add(T q, float sigma, float c) { return fmaf(widen(q), sigma, c); }
  template <bool SPLIT = false>
  __device__ __forceinline__ static float decode_sub(T q, float sigma, float c) { return fmaf(widen(q), -sigma, c); }
  // the gfx950 conversion (one instruction where rounding by hand took three:
  // 512^3 2710 -> 2686 us a step, 130 x 50 x 70 11.9 -> 11.6)
  __device__ __forceinline__ static T encode(float d, float inv_sigma) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(d * inv_sigma));
  }
};

// Byte size of one stored value.
constexpr int storage_bytes(int s) { return s == kF32 ? 4 : 2; }

// A stored element as a 32-bit word (16-bit types zero-extended) and back.
template <class T>
__device__ __forceinline__ uint32_t to_bits(T q) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(uint32_t, q);
  else return __builtin_bit_cast(uint16_t, q);
}
template <class T>
__device__ __forceinline__ T from_bits(uint32_t b) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, b);
  else return __builtin_bit_cast(T, static_cast<uint16_t>(b));
}

// Periodic neighbour coordinate: c in {-1, 0, 1}.
__host__ __device__ __forceinline__ uint32_t wrap_add(uint32_t x, int c, uint32_t n) {
  return c == 0 ? x : (c > 0 ? (x + 1 == n ? 0u : x + 1) : (x == 0 ? n - 1 : x - 1));
}

}  // namespace rflbm
