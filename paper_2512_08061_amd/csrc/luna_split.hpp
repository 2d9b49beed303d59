// luna_split.hpp -- products of fp32 operands with bf16 ones on the bf16 matrix cores.
//
// An fp32 value is the sum of three bf16 ones (to 2^-24 of it), so its product with a
// bf16 value is three bf16 matrix-core products accumulated in fp32: as exact as the fp32
// matrix cores, at a fifth of their time (3 x 16 cycles per 16 x 16 x 32 block against
// 8 x 32).  Two fp32 operands stay on the fp32 matrix cores.
#pragma once

#include "luna_device.hpp"

namespace luna {

struct Split3 {
  Frag<__bf16> p[3];
};
__device__ __forceinline__ void split3(Split3& s, const float (&x)[8]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e % 2 == 0) s.p[k].set2(e, r[e], r[e + 1]);
      const float h = s.p[k].get(e);
      if (k == 0) r[e] = r[e] == h ? 0.0f : r[e] - h;  // (an infinity is its first part alone)
      else if (k == 1) r[e] -= h;
    }
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
