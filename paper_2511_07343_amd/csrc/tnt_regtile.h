// Register-resident MFMA tiles as operands (gfx950, bf16 16x16x32).
//
// An accumulator tile holds rows 4(l/16)+r, r = 0..3, of column l%16 in lane
// l.  Two such tiles stacked along the contraction (rows k0..k0+15 and
// k0+16..k0+31) give lane l the contraction indices k0+4(l/16)+r and
// k0+16+4(l/16)+r, one B operand of v_mfma_f32_16x16x32_bf16 whose 32 slots
// are summed in any order: the A operand only has to present the same index in
// the same slot, i.e. two 8-byte reads at k0+4(l/16) and k0+16+4(l/16) of a
// contraction-contiguous row (a_pair) instead of one 16-byte read.  A tile
// used this way contracts over its row index.
#pragma once

#include "tnt_device.h"

namespace tnt {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The wave's index as a wave-uniform (scalar) value, so that everything
// derived from it stays in scalar registers.
__device__ __forceinline__ int wave_id_uniform() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
}

__device__ __forceinline__ bf16x4 cvt4(const f4& a) {
  bf16x4 b;
  b[0] = (__bf16)a[0]; b[1] = (__bf16)a[1]; b[2] = (__bf16)a[2]; b[3] = (__bf16)a[3];
  return b;
}

__device__ __forceinline__ bf16x8 join(const bf16x4& a, const bf16x4& b) {
  bf16x8 f;
  f[0] = a[0]; f[1] = a[1]; f[2] = a[2]; f[3] = a[3];
  f[4] = b[0]; f[5] = b[1]; f[6] = b[2]; f[7] = b[3];
  return f;
}

__device__ __forceinline__ bf16x4 zero_bf4() {
  bf16x4 z;
  z[0] = z[1] = z[2] = z[3] = (__bf16)0.0f;
  return z;
}

// A operand row `row` of a contraction-contiguous array (LDS or global),
// contraction indices k0 + 4g + j and k0 + 16 + 4g + j (j = 0..3), matching a
// B operand made of two stacked accumulator tiles; `hi` = false zero-fills the
// second half (a contraction of 16).
__device__ __forceinline__ bf16x8 a_pair(const __bf16* A, int ld, int row, int k0, int g,
                                         bool hi = true) {
  // a 32-bit element offset from the (wave-uniform) base: scalar base + vector
  // offset addressing, one address register per load instead of a pair
  const __bf16* p = A + (uint32_t)(row * ld + k0 + 4 * g);
  const bf16x4 x = *reinterpret_cast<const bf16x4*>(p);
  const bf16x4 y = hi ? *reinterpret_cast<const bf16x4*>(p + 16) : zero_bf4();
  return join(x, y);
}

// A float's bits 8 to 15, the byte that follows its bf16 value, of four floats in a word.
// Beside the bf16 value they give the float back to 2^-17 of itself: the byte as a signed
// one counts from the rounded value (which lies above the float where the byte's top bit
// is set; a float half way between two bf16 values, 1 in 2^16, comes back one off).
__device__ __forceinline__ unsigned rem_pack(const f4& x) {
  const float a = x[0], b = x[1], c = x[2], d = x[3];
  const unsigned lo = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, b), __builtin_bit_cast(unsigned, a), 0x0c0c0501u);
  const unsigned hi = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, d), __builtin_bit_cast(unsigned, c), 0x05010c0cu);
  return lo | hi;
}
__device__ __forceinline__ f4 rem_unpack(const bf16x4& hi, unsigned w) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const u2 h = __builtin_bit_cast(u2, hi);
  f4 x;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const unsigned top = r % 2 ? (h[r / 2] & 0xffff0000u) : (h[r / 2] << 16);
    const int q = (int)(w << (24 - 8 * r)) >> 24;
    const unsigned bits = (top | 0x80u) + ((unsigned)q << 8);
    x[r] = __builtin_bit_cast(float, bits);
  }
  return x;
}
// The remainders of a state in words of two (W and S): first those of W1, S1, then (after
// hid d / 4) of W2, S2, a 16 x 16 tile (d tile dt of nd, hidden tile ht) in the order of
// the lanes that hold it: of W1, S1 lane l has hidden rows 4 (l / 16) .. + 3 of column
// l % 16 of d, of W2, S2 rows 4 (l / 16) .. + 3 of d of hidden column l % 16.  A store or
// load of a tile is one run of 512 bytes (by matrix rows, stores of 32-byte pieces cost
// the forward walk 3.5 us a chunk).
typedef unsigned rem2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t rem_ofs(int nd, int dt, int ht, int l) {
  return (uint32_t)((ht * nd + dt) * 64 + l);
}
// the lane that holds, of W1, the values that lane l of the transposed tile has after a
// transpose within its quad
__device__ __forceinline__ int rem_lane1(int l) { return (l & 12) * 4 + (l >> 4) * 4 + (l & 3); }

__device__ __forceinline__ void mma32(f4& acc, const bf16x8& a, const bf16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

}  // namespace tnt
