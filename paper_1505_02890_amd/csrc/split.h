// fp32 products on the bf16 matrix cores.
//
// A float splits into three bf16 values, a = h + m + l: h is a rounded to
// bf16, m the rest rounded, l the rest of that; 3 x 8 significant bits hold
// all 24 of a (exactly, down to |a| = 2^-109; bf16 has no bits below 2^-133).
// Six of the nine products of two such numbers,
//   a b = hh' + (hm' + mh') + (hl' + mm' + lh') + rest,
// each exact in fp32 and summed in fp32 by the matrix core, stand for one
// fp32 product.  The rest is at most 2^-24 |a b|, half an fp32 ulp, and 2^-26.5
// as rms over random mantissas.  Six bf16 instructions cost 6/16 of the fp32
// instruction for the same product (v_mfma_f32_32x32x16_bf16 against
// v_mfma_f32_16x16x4f32: 2190 against 141 TFLOP/s in a register-only loop, so
// 365 against 141 effective), and their sums round once per 16 products instead
// of once per 4: on N(0, 1) operands the error against 64-bit sums is 1.1e-7 /
// 3.1e-7 / 6.3e-7 for 64 / 384 / 1728 products, 1.5e-7 / 3.6e-7 / 7.5e-7 on
// the fp32 instruction.
//
// Operands that the split cannot hold are found after the fact, and the sums
// that they enter are redone on the fp32 instruction:
//  - An infinity, a NaN or a value that rounds past bf16's largest turns the
//    rests into NaN, so every sum it enters is NaN or infinite.
//  - Values below 2^-109 lose what lies below 2^-133.  That counts where
//    nothing larger stands beside them: an operand row whose largest value is
//    below 2^-95 (tiny) is redone.  The tile kernels see it by a row's sums, none
//    of which can then exceed its column's sum |W| 2^-95, and columns of tiny
//    weights when they are packed; the weight gradient watches its operands
//    (Seen).  (Watching them in the tile kernels' loops too cost 1 to 3%, or with
//    Seen's branch, which spills there, all of the time again.)  Beside a
//    value of 2^-95 or more the loss is below 2^-38 of it.  (Rows with nothing
//    above 2^-134 have no high parts and are taken as zero.)
#pragma once

#include <hip/hip_runtime.h>

namespace scn {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f_ __attribute__((ext_vector_type(2)));
typedef __bf16 v2b_ __attribute__((ext_vector_type(2)));
typedef __bf16 v8b_ __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// two floats rounded to bf16, the first in the low half
__device__ inline uint32_t cvt2_bf16(float a, float b) {
  const v2f_ v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2b_));
}

__device__ inline void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = cvt2_bf16(a, b);
  const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
  m = cvt2_bf16(ra, rb);
  const float sa = ra - __uint_as_float(m << 16), sb = rb - __uint_as_float(m & 0xffff0000u);
  l = cvt2_bf16(sa, sb);
}

// What a 32-row operand tile has held so far, a bit per lane (lanes r and 32 + r
// hold row r): values but zero, and values of at least 2^-95 (an exponent of 32
// and more has one of the top three exponent bits).  Both live in scalar
// registers, and once every lane has held a large value there is no more to see.
__device__ inline uint32_t or_bits(uint32_t o, v4u h) { return o | h[0] | h[1] | h[2] | h[3]; }
struct Seen {
  uint64_t any = 0, big = 0;
  __device__ inline void add(v4u h) {
    if (big != ~0ull) {
      const uint32_t o = or_bits(0, h);
      any |= __ballot((o & 0x7fff7fffu) != 0);
      big |= __ballot((o & 0x70007000u) != 0);
    }
  }
  // rows that have held something, and something large
  __device__ inline uint32_t any32() const { return (uint32_t)(any | any >> 32); }
  __device__ inline uint32_t big32() const { return (uint32_t)(big | big >> 32); }
};

// Whether the bits of floats, or'ed together, say the same of them: not all
// zero, and none of 2^-95 or more.
__device__ inline bool tiny_floats(uint32_t o) {
  return (o & 0x7fffffffu) != 0 && (o & 0x70000000u) == 0;
}

// One MFMA operand of eight values along the reduction: s[0] high, s[1]
// middle, s[2] low parts.
struct Frag3 {
  v4u s[3];
};

__device__ inline Frag3 split8(const float (&v)[8]) {
  Frag3 f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t h, m, l;
    split2(v[2 * j], v[2 * j + 1], h, m, l);
    f.s[0][j] = h;
    f.s[1][j] = m;
    f.s[2][j] = l;
  }
  return f;
}

__device__ inline v16f mfma_bf16(v4u a, v4u b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b_, a),
                                                 __builtin_bit_cast(v8b_, b), c, 0, 0, 0);
}

// the six products, smallest first
constexpr int SPLIT_PROD = 6;
__device__ constexpr int split_a(int p) { return p == 0 ? 0 : p == 1 ? 2 : p == 2 ? 1 : p == 3 ? 0 : p == 4 ? 1 : 0; }
__device__ constexpr int split_b(int p) { return p == 0 ? 2 : p == 1 ? 0 : p == 2 ? 1 : p == 3 ? 1 : p == 4 ? 0 : 0; }

}  // namespace scn
