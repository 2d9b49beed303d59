// luna_split.hpp -- products of fp32 operands with bf16 ones on the bf16 matrix cores.
//
// An fp32 value is the sum of three bf16 ones (to 2^-24 of it), so its product with a
// bf16 value is three bf16 matrix-core products accumulated in fp32: as exact as the fp32
// matrix cores, at a fifth of their time (3 x 16 cycles per 16 x 16 x 32 block against
// 8 x 32).  Two fp32 operands stay on the fp32 matrix cores.
//
// Every fp32 value may be split, an infinity too.  The bf16 one has to be finite, or to meet
// the first part alone: beside the others an infinity would give infinities of either sign or
// NaN where its fp32 product is infinite.
#pragma once

#include "luna_device.hpp"

namespace luna {

constexpr float kBf16Max = 0x1.fep127f;

struct Split3 {
  Frag<__bf16> p[3];
};
// ALL: also values above kBf16Max, whose first part would be infinite (the others then cancel
// it to NaN); two more instructions per pair.
template <bool ALL = true>
__device__ __forceinline__ void split3(Split3& s, const float (&x)[8]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
  float most = kBf16Max;
  asm("" : "+s"(most));  // (one scalar register for both bounds: two constants take vector registers)
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e % 2 == 0) {
        if (ALL && k == 0)
          s.p[k].set2(e, __builtin_amdgcn_fmed3f(r[e], -most, most), __builtin_amdgcn_fmed3f(r[e + 1], -most, most));
        else s.p[k].set2(e, r[e], r[e + 1]);
      }
      const float h = s.p[k].get(e);
      // (an infinity is its first part alone, or its second beside kBf16Max)
      if (k == (ALL ? 1 : 0)) r[e] = r[e] == h ? 0.0f : r[e] - h;
      else if (k < 2) r[e] -= h;
    }
}

__device__ __forceinline__ Frag<float> widen(const Frag<__bf16>& f) {
  Frag<float> w;
#pragma unroll
  for (int e = 0; e < 8; ++e) w.v[e] = f.get(e);
  return w;
}
__device__ __forceinline__ Frag<float> widen(const Frag<float>& f) { return f; }

// whether a bf16 value beside a split operand is infinite or NaN (fp32 ones meet no parts)
__device__ __forceinline__ bool not_finite(const Frag<__bf16>& f) {
  typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
  const i32x4 w = __builtin_bit_cast(i32x4, f.v);
  u16x2 m = {0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[i] & 0x7fff7fff));
  return m[0] >= 0x7f80 || m[1] >= 0x7f80;
}
// infinities and NaN as 1 of their sign: the products with the second and third part of a
// split operand that then go with those with its first
__device__ __forceinline__ void to_ones(Frag<__bf16>& f) {
  i32x4 w = __builtin_bit_cast(i32x4, f.v);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if ((w[i] & 0x7f80) == 0x7f80) w[i] = (w[i] & 0xffff8000) | 0x3f80;
    if ((w[i] & 0x7f800000) == 0x7f800000) w[i] = (w[i] & 0x8000ffff) | 0x3f800000;
  }
  f.v = __builtin_bit_cast(bf16x8, w);
}

// c += a x and c += x b for an fp32 operand x split in three
__device__ __forceinline__ void mma(f32x4& c, const Frag<__bf16>& a, const Split3& x) {
#pragma unroll
  for (int k = 2; k >= 0; --k) mma(c, a, x.p[k]);
}
__device__ __forceinline__ void mma(f32x4& c, const Split3& x, const Frag<__bf16>& b) {
#pragma unroll
  for (int k = 2; k >= 0; --k) mma(c, x.p[k], b);
}

// The form an operand of type X takes next to one of type Y.
template <typename X, typename Y>
struct OperandOf {
  using type = Frag<X>;
};
template <>
struct OperandOf<float, __bf16> {
  using type = Split3;
};
template <typename X, typename Y>
using Operand = typename OperandOf<X, Y>::type;

template <typename X>
__device__ __forceinline__ void set_operand(Frag<X>& o, const Frag<X>& f) { o = f; }
__device__ __forceinline__ void set_operand(Split3& o, const Frag<float>& f) { split3(o, f.v); }

}  // namespace luna
