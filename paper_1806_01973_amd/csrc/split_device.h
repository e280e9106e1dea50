// fp32 operands on the bf16 matrix cores: x = h + m + l exactly, each part the
// bf16 rounding of what the parts before it leave (8 + 8 + 8 significand bits
// hold fp32's 24).
#pragma once

#include "device_util.h"

namespace pinsage {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct Split3 {
  u32x4 p[3];
};

// The eight products of parts that reach fp32's last bits, as (part of b, part of
// a), smallest first: (2,1) (1,2) (2,0) (0,2) (1,1) (1,0) (0,1) (0,0). The one left
// out is at most 2^-34 of a product of powers of two, below 2^-33 of any; without
// (2,1) and (1,2) a lone product was off by up to 1.9 * 2^-25 before its rounding.
constexpr int kSplitProducts = 8;
__device__ constexpr int split_b(int t) {
  return t == 0 || t == 2 ? 2 : (t == 1 || t == 4 || t == 5 ? 1 : 0);
}
__device__ constexpr int split_a(int t) {
  return t == 1 || t == 3 ? 2 : (t == 0 || t == 4 || t == 6 ? 1 : 0);
}

// What the parts cover. A value's lowest bit lies 23 binary places below its
// leading one, and bf16 ends at 2^-133 (the matrix cores keep its subnormals), so
// the parts of values below 2^-110 lose bits; and products of parts end at 2^-149,
// 46 places below the leading product's own first bit. A pair of operands is
// covered when both are at least 2^-110 and their product at least 2^-100.
// Magnitudes are kept as keys 2 |x| - 1 of the bit patterns: ordered like |x| but
// for zero, which is above everything (a zero is always covered); bits 24 .. 31 are
// the biased exponent, or one less for a power of two.
__device__ __forceinline__ uint32_t magnitude_key(uint32_t bits) { return (bits << 1) - 1u; }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t least_key(const u32x4& u, const u32x4& v, uint32_t key) {
#pragma unroll
  for (int q = 0; q < 4; ++q) key = umin(umin(magnitude_key(u[q]), magnitude_key(v[q])), key);
  return key;
}
__device__ __forceinline__ uint32_t wave_min_key(uint32_t key) {  // bit 0 lost
  return ~((uint32_t)wave_max_i32((int)(~key >> 1)) << 1);
}
__device__ __forceinline__ bool split_covers(uint32_t key_a, uint32_t key_b) {
  const uint32_t ea = key_a >> 24, eb = key_b >> 24;
  return ea >= 127 - 110 && eb >= 127 - 110 && ea + eb >= 254 - 100;
}

// Parts of the eight fp32 values u[0..3], v[0..3]; key: the least magnitude key so far.
__device__ __forceinline__ Split3 split3(const u32x4& u, const u32x4& v, uint32_t& key) {
  Split3 s;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t u0 = q < 2 ? u[2 * q] : v[2 * q - 4], u1 = q < 2 ? u[2 * q + 1] : v[2 * q - 3];
    key = umin(umin(magnitude_key(u0), magnitude_key(u1)), key);
    float x0 = __uint_as_float(u0), x1 = __uint_as_float(u1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const uint32_t w = pack_bf16x2(x0, x1);
      s.p[t][q] = w;
      if (t < 2) {
        x0 -= __uint_as_float(w << 16);
        x1 -= __uint_as_float(w & 0xFFFF0000u);
      }
    }
  }
  return s;
}

}  // namespace pinsage
