// luna_chunk_kernel.hpp -- the chunked attention kernel behind luna_chunk.hpp.
//
// A workgroup of eight waves owns 64 tokens ("rows") of a head.  With S, z the state outside
// its piece (or the total), x, y the features and u, v the values of rows and columns:
//
//   query pass  num = x S + P v,  P = tril(x y^T),  den = x z + P 1 + eps
//               forward: out = num / den, else with w = 1 / den, e = -(u . num) w^2
//               dx = w (u S^T) + e z + R y,  R = tril(w (u v^T) + e)
//   key pass    dv = x S + P v with P = (x y^T) w over the queries at or after each key,
//               dx = u S^T + z + R y,  R = (u v^T) w + e likewise (w, e of the queries)
//
// All products run transposed (output columns as the A operand, rows as the B operand), so
// that a lane ends with four consecutive outputs of one token.  Two fp32 operands meet on the
// fp32 matrix cores, an fp32 and a bf16 one as three bf16 products (luna_split.hpp); row
// features, row values and P or R wait in LDS, the operands from memory are read by one wave
// each, for up to four row blocks, and asked for a phase or a barrier before their use.
//
// Bound by the fp32 matrix cores and by the barriers between the phases of the one or two
// workgroups that a compute unit holds.  Backward of 32 x 12 heads of 512 tokens, d = D = 64:
// 58 + 56 us for the two passes, where the fp32 GEMMs on tiles padded from 65 columns, the
// packing of [V | 1] and the conversions took 345; causal, 2 x 16 heads of 2048 tokens,
// d = 128, D = 256: 205 + 196 us instead of 790.  Causal forward of 2 x 16 heads of 1024 fp32
// tokens, D = 128: 36 us instead of 115.
#pragma once

#include <algorithm>

#include "luna_chunk.hpp"
#include "luna_device.hpp"
#include "luna_split.hpp"

namespace luna {

namespace {

constexpr int kCkThreads = 512;
constexpr int kPassQuery = 0, kPassKey = 1;

// Everything is read through range-checked buffers that end with the operand's last row, so
// that rows past it read as 0: a test per load would put a branch around each (measured: the
// kernel takes twice the time).

// 8 floats of row t of a [.][len] array at k0, 0 past the row's end (vec: len is a multiple of 8)
__device__ __forceinline__ void row8(float (&o)[8], Buf b, int t, int k0, int len, bool vec) {
  const int off = (t * len + k0) * 4;
  if (vec) {
    Frag<float> f;
    buf_load8(f, b, k0 < len ? off : kPastEnd);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = f.v[e];
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      o[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, k0 + e < len ? off + 4 * e : kPastEnd, 0, 0));
  }
}
__device__ __forceinline__ void to_frag(Frag<float>& f, const float (&x)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) f.v[e] = x[e];
}
// 8 elements `stride` apart from element `at`
__device__ __forceinline__ void col8(float (&o)[8], Buf b, int at, int stride) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    o[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (at + e * stride) * 4, 0, 0));
}
__device__ __forceinline__ void col8(Frag<float>& f, Buf b, int at, int stride) {
  float x[8];
  col8(x, b, at, stride);
  to_frag(f, x);
}
__device__ __forceinline__ void col8(Frag<__bf16>& f, Buf b, int at, int stride) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    f.v[e] = __builtin_bit_cast(__bf16, __builtin_amdgcn_raw_buffer_load_b16(b, (at + e * stride) * 2, 0, 0));
}

// c + lo += a b of a value and an fp32 operand: the small parts of a split operand gather in
// `lo`, fp32 products all do, so that they are not rounded one by one at the size of c.
__device__ __forceinline__ void mma_value(f32x4&, f32x4& lo, const Frag<float>& a, const Frag<float>& b) {
  mma(lo, a, b);
}
__device__ __forceinline__ void mma_value(f32x4& c, f32x4& lo, const Split3& a, const Frag<__bf16>& b) {
  mma(lo, a.p[2], b);
  mma(lo, a.p[1], b);
  mma(c, a.p[0], b);
}

// P in LDS as the other operand of a value: split in bf16 planes, or fp32
__device__ __forceinline__ void put_p(const f32x4& p, __bf16* dst, int plane) {
  float x[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = p[j], x[4 + j] = 0.0f;
  Split3 s;
  split3(s, x);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    bf16x4 h;
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = s.p[k].v[j];
    *reinterpret_cast<bf16x4*>(dst + k * plane) = h;
  }
}
__device__ __forceinline__ void put_p(const f32x4& p, float* dst, int) { *reinterpret_cast<f32x4*>(dst) = p; }

// KB: 32-feature steps held (D <= 32 KB)
template <typename T, int DH, int KB>
struct CkCfg {
  static constexpr int DK = 32 * KB, LDX = DK + 4, LDU = DH + 16 / (int)sizeof(T);
  static constexpr int LDP = kChunkTile + 16 / (int)sizeof(T), LDR = kChunkTile + 4;
  static constexpr int PP = kChunkTile * LDP;  // a plane of P (elements)
  static constexpr size_t XB = (size_t)kChunkTile * LDX * 4, UB = (size_t)kChunkTile * LDU * sizeof(T);
  static constexpr size_t PB = sizeof(T) == 2 ? (size_t)3 * PP * 2 : (size_t)PP * 4;  // (R: fp32, less)
  static constexpr size_t SB = ((size_t)(4 + 8 + 5) * kChunkTile + DK) * 4;
  static constexpr size_t lds(bool causal, bool grads) { return XB + SB + (grads ? UB : 0) + (causal ? PB : 0); }
  static_assert(PB >= (size_t)kChunkTile * LDR * 4, "R takes the place of P");
};

template <typename T, int DH, int KB, int PASS>
__global__ __launch_bounds__(kCkThreads, KB <= 4 ? 4 : 2) void chunk_kernel(ChunkArgs a) {
  using C = CkCfg<T, DH, KB>;
  using SOp = Operand<float, T>;  // an fp32 operand next to a value
  constexpr int LDX = C::LDX, LDU = C::LDU, LDP = C::LDP, LDR = C::LDR, PP = C::PP;
  constexpr int CB = DH / 16, CBW = CB < 8 ? CB : 8;  // value blocks: one per wave,
  constexpr int R1 = 4 * CBW / 8;                     // for R1 of the four row blocks
  constexpr int FPW = KB > 4 ? KB / 4 : 1;            // feature blocks per wave,
  constexpr int R2 = KB >= 4 ? 4 : 2;                 // for R2 of the four row blocks
  constexpr int FBW = KB >= 4 ? 8 : 4;                // feature blocks met in one go
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* xs = reinterpret_cast<float*>(lds);                  // row features
  float* denp = reinterpret_cast<float*>(lds + C::XB);        // [4][64] row sums of P per column block
  float* dots = denp + 4 * kChunkTile;                        // [8][64]
  float* deni = dots + 8 * kChunkTile;                        // x z
  float* wr = deni + kChunkTile;                              // rows: w, e (query pass)
  float* wc = wr + 2 * kChunkTile;                            // columns: w, e (key pass)
  float* zs = wc + 2 * kChunkTile;                            // z (query pass)
  const bool grads = PASS == kPassKey || a.u != nullptr;
  T* us = reinterpret_cast<T*>(lds + C::XB + C::SB);          // row values (with gradients)
  T* ps = reinterpret_cast<T*>(lds + C::XB + C::SB + (grads ? C::UB : 0));  // P: [row][column]
  float* rs = reinterpret_cast<float*>(ps);                   // then R
  const int tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int g = lane / 16, r = lane % 16;
  // neighbouring tiles share states and columns: consecutive ones on one die (eight dies,
  // workgroups dealt to them in turn)
  const unsigned per = gridDim.x / 8, extra = gridDim.x % 8, die = blockIdx.x % 8;
  const unsigned id = die * per + min(die, extra) + blockIdx.x / 8;
  const int tiles = (int)((a.n + kChunkTile - 1) / kChunkTile);
  const unsigned launched = (unsigned)((tiles - a.first + a.step - 1) / a.step);  // of every head
  const int64_t head = id / launched;
  const int tile = a.first + a.step * (int)(id - (unsigned)head * launched);
  const int64_t t0 = (int64_t)tile * kChunkTile;
  const int rows = (int)min((int64_t)kChunkTile, a.n - t0);
  const int D = a.D, kbs = (D + 31) / 32, tpp = a.piece / kChunkTile;
  const bool vec = D % 8 == 0;  // (uniform) feature rows are whole 32-byte pieces
  const int piece = tile / tpp;
  // column tiles of the piece on this tile's side of the diagonal
  const int c_first = !a.causal ? 0 : PASS == kPassQuery ? piece * tpp : tile;
  const int c_end = !a.causal ? 0 : PASS == kPassQuery ? tile + 1 : min(tiles, (piece + 1) * tpp);
  const float* S = a.state + (head * a.pieces + (a.causal ? piece : 0)) * a.elems;
  const float* z = S + (int64_t)D * DH;
  const Buf bS = buffer(S, D * DH * 4);
  const Buf bx = buffer(a.x + (head * a.n + t0) * D, rows * D * 4);
  const Buf bu = buffer(reinterpret_cast<const T*>(a.u) + (head * a.n + t0) * DH, rows * DH * (int)sizeof(T));
  auto cols_of = [&](int ct) { return (int)min((int64_t)kChunkTile, a.n - (int64_t)ct * kChunkTile); };
  auto y_of = [&](int ct) {
    return buffer(a.y + (head * a.n + (int64_t)ct * kChunkTile) * D, cols_of(ct) * D * 4);
  };
  auto v_of = [&](int ct) {
    return buffer(reinterpret_cast<const T*>(a.v) + (head * a.n + (int64_t)ct * kChunkTile) * DH,
                  cols_of(ct) * DH * (int)sizeof(T));
  };

  // ---- x S, and x z spread over the first four waves
  const int cb = wave % CBW, rb1 = wave / CBW * R1;
  const bool dwave = PASS == kPassQuery && wave < 4;
  float sn[KB][8];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) col8(sn[kb], bS, (32 * kb + 8 * g) * DH + 16 * cb + r, DH);
  {
    constexpr int XI = kChunkTile * 4 * KB / kCkThreads, UI = kChunkTile * DH / 8 / kCkThreads;
    float f[XI][8];
    Frag<T> uf[UI > 0 ? UI : 1];
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      const int c = tid + kCkThreads * i;
      row8(f[i], bx, c / (4 * KB), 8 * (c % (4 * KB)), D, vec);
    }
    if (grads) {
#pragma unroll
      for (int i = 0; i < (UI > 0 ? UI : 1); ++i) {
        buf_load8(uf[i], bu, (tid + kCkThreads * i) * 8 * (int)sizeof(T));
      }
    }
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      const int c = tid + kCkThreads * i;
      Frag<float> ff;
      to_frag(ff, f[i]);
      store8(xs + c / (4 * KB) * LDX + 8 * (c % (4 * KB)), ff);
    }
    if (grads) {
#pragma unroll
      for (int i = 0; i < (UI > 0 ? UI : 1); ++i) {
        const int c = tid + kCkThreads * i;
        if (UI > 0 || c < kChunkTile * DH / 8) store8(us + c / (DH / 8) * LDU + 8 * (c % (DH / 8)), uf[i]);
      }
    }
  }
  if (PASS == kPassQuery) {
    if (tid < 4 * kChunkTile) denp[tid] = 0.0f;
    if (tid < C::DK) zs[tid] = tid < D ? z[tid] : 0.0f;
  }
  __syncthreads();
  f32x4 num[R1], lo1[R1];
#pragma unroll
  for (int b = 0; b < R1; ++b) num[b] = lo1[b] = zero4();
  // this wave's block of P: column block sc of a tile, row blocks sr and sr + 1
  const int sc = wave % 4, sr = wave / 4 * 2;
  float yn[KB][8];
  auto load_y = [&](Buf by, int kb) { row8(yn[kb], by, 16 * sc + r, 32 * kb + 8 * g, D, vec); };
  {
    f32x4 den = zero4();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (kb > 0 && kb >= kbs) break;  // (uniform)
      Frag<float> sa;
      to_frag(sa, sn[kb]);
      if (c_first < c_end) load_y(y_of(c_first), kb);
#pragma unroll
      for (int b = 0; b < R1; ++b) {
        Frag<float> xb;
        load8(xb, xs + (16 * (rb1 + b) + r) * LDX + 32 * kb + 8 * g);
        mma(num[b], sa, xb);
      }
      if (dwave) {
        Frag<float> xb, za;
        load8(xb, xs + (16 * wave + r) * LDX + 32 * kb + 8 * g);
        load8(za, zs + 32 * kb + 8 * g);
        mma(den, za, xb);
      }
    }
    if (dwave && g == 0) deni[16 * wave + r] = den[0];
  }

  // pair (column 16 sc + 4 g + j, row 16 (sr + b) + r) of column tile ct is on the far side
  // of the diagonal
  auto masked = [&](int ct, int b, int j) {
    const int col = 16 * sc + 4 * g + j, row = 16 * (sr + b) + r;
    return ct == tile && (PASS == kPassQuery ? col > row : col < row);
  };
  auto load_wc = [&](int ct) {
    if (PASS == kPassKey && tid < kChunkTile) {
      const int64_t t = (int64_t)ct * kChunkTile + tid;
      const bool ok = t < a.n;
      wc[tid] = ok ? a.w[(head * a.n + t) * 2] : 0.0f;
      wc[kChunkTile + tid] = ok ? a.w[(head * a.n + t) * 2 + 1] : 0.0f;
    }
  };

  // ---- + P v
  for (int ct = c_first; ct < c_end; ++ct) {
    const int cols = cols_of(ct);
    const Buf bv = v_of(ct);
    load_wc(ct);
    Frag<T> va[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) col8(va[ks], bv, (32 * ks + 8 * g) * DH + 16 * cb + r, DH);
    f32x4 p[2];
    p[0] = zero4();
    p[1] = zero4();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (kb > 0 && kb >= kbs) break;  // (uniform)
      Frag<float> ya;
      to_frag(ya, yn[kb]);
      if (ct + 1 < c_end) load_y(y_of(ct + 1), kb);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        Frag<float> xb;
        load8(xb, xs + (16 * (sr + b) + r) * LDX + 32 * kb + 8 * g);
        mma(p[b], ya, xb);
      }
    }
    __syncthreads();  // the last tile's P is no longer read; wc is written
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (PASS == kPassKey) p[b][j] *= wc[16 * sc + 4 * g + j];
        if (masked(ct, b, j) || 16 * sc + 4 * g + j >= cols) p[b][j] = 0.0f;
      }
      if (PASS == kPassQuery) {
        float s = (p[b][0] + p[b][1]) + (p[b][2] + p[b][3]);
        s += __shfl_xor(s, 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (g == 0) denp[sc * kChunkTile + 16 * (sr + b) + r] += s;
      }
      put_p(p[b], ps + (16 * (sr + b) + r) * LDP + 16 * sc + 4 * g, PP);
    }
    __syncthreads();
    auto p_of = [&](int ks, int b, int k) {
      Frag<T> p;
      load8(p, ps + k * PP + (16 * (rb1 + b) + r) * LDP + 32 * ks + 8 * g);
      return p;
    };
    if constexpr (sizeof(T) == 2) {  // (the parts gather as in mma_value)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int b = 0; b < R1; ++b) mma(num[b], va[ks], p_of(ks, b, 0));
        if (__any(not_finite(va[ks]))) to_ones(va[ks]);  // (uniform)
#pragma unroll
        for (int b = 0; b < R1; ++b) {
          mma(lo1[b], va[ks], p_of(ks, b, 2));
          mma(lo1[b], va[ks], p_of(ks, b, 1));
        }
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int b = 0; b < R1; ++b) mma(lo1[b], va[ks], p_of(ks, b, 0));
    }
  }
#pragma unroll
  for (int b = 0; b < R1; ++b) num[b] += lo1[b];

  // this wave's feature blocks of dx and their operands
  const int fb = wave % FBW, rb2 = wave / FBW * R2;
  float s8[DH / 32][FPW][8], zf[FPW][4];
  if (grads) {
#pragma unroll
    for (int f = 0; f < FPW; ++f) {
      const int ft = 16 * (fb + 8 * f);
#pragma unroll
      for (int kc = 0; kc < DH / 32; ++kc)
        row8(s8[kc][f], bS, ft + r, 32 * kc + 8 * g, DH, true);
#pragma unroll
      for (int j = 0; j < 4; ++j) zf[f][j] = ft + 4 * g + j < D ? z[ft + 4 * g + j] : 0.0f;
    }
  }

  if (PASS == kPassKey) {
    if (!a.dx) __syncthreads();  // (dV in the place of dO: every wave has its columns)
    T* out = reinterpret_cast<T*>(a.out) + (head * a.n + t0) * DH;
#pragma unroll
    for (int b = 0; b < R1; ++b) {
      const int t = 16 * (rb1 + b) + r;
      if (a.out && t < rows) store4(out + (int64_t)t * DH + 16 * cb + 4 * g, num[b][0], num[b][1], num[b][2], num[b][3]);
    }
    if (!a.dx) return;
  } else {
    if (grads)
#pragma unroll
      for (int b = 0; b < R1; ++b) {
        const int t = 16 * (rb1 + b) + r;
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) s = fmaf((float)us[t * LDU + 16 * cb + 4 * g + j], num[b][j], s);
        s += __shfl_xor(s, 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (g == 0) dots[cb * kChunkTile + t] = s;
      }
    __syncthreads();  // deni, denp, dots
    auto den_of = [&](int t) {
      return deni[t] + ((denp[t] + denp[64 + t]) + (denp[128 + t] + denp[192 + t])) + a.eps;
    };
    if (!grads) {
      T* out = reinterpret_cast<T*>(a.out) + (head * a.n + t0) * DH;
#pragma unroll
      for (int b = 0; b < R1; ++b) {
        const int t = 16 * (rb1 + b) + r;
        const float inv = 1.0f / den_of(t);
        if (t < rows)
          store4(out + (int64_t)t * DH + 16 * cb + 4 * g, num[b][0] * inv, num[b][1] * inv, num[b][2] * inv,
                 num[b][3] * inv);
      }
      return;
    }
    if (tid < kChunkTile) {
      float dot = 0.0f;
#pragma unroll
      for (int k = 0; k < CBW; ++k) dot += dots[k * kChunkTile + tid];
      const float inv = 1.0f / den_of(tid);
      const bool ok = tid < rows;
      const float w = ok ? inv : 0.0f, e = ok ? -dot * inv * inv : 0.0f;
      wr[tid] = w;
      wr[kChunkTile + tid] = e;
      if (ok) {
        a.w[(head * a.n + t0 + tid) * 2] = w;
        a.w[(head * a.n + t0 + tid) * 2 + 1] = e;
      }
    }
  }

  // ---- u S^T
  f32x4 acc[FPW][R2], lo2[FPW][R2];
#pragma unroll
  for (int f = 0; f < FPW; ++f)
#pragma unroll
    for (int b = 0; b < R2; ++b) acc[f][b] = lo2[f][b] = zero4();
#pragma unroll
  for (int kc = 0; kc < DH / 32; ++kc) {
    SOp sa[FPW];
#pragma unroll
    for (int f = 0; f < FPW; ++f) {
      Frag<float> t;
      to_frag(t, s8[kc][f]);
      set_operand(sa[f], t);
    }
#pragma unroll
    for (int b = 0; b < R2; ++b) {
      Frag<T> ub;
      load8(ub, us + (16 * (rb2 + b) + r) * LDU + 32 * kc + 8 * g);
#pragma unroll
      for (int f = 0; f < FPW; ++f) mma_value(acc[f][b], lo2[f][b], sa[f], ub);
    }
  }
  Frag<T> vr[DH / 32];
  float y8[2][FPW][8];
  auto load_ry = [&](int ct) {
    const Buf by = y_of(ct), bv = v_of(ct);
#pragma unroll
    for (int kc = 0; kc < DH / 32; ++kc)
      buf_load8(vr[kc], bv, ((16 * sc + r) * DH + 32 * kc + 8 * g) * (int)sizeof(T));
    // (features past D only meet accumulator rows that are not stored)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int f = 0; f < FPW; ++f) col8(y8[ks][f], by, (32 * ks + 8 * g) * D + 16 * (fb + 8 * f) + r, D);
  };
  if (c_first < c_end) load_ry(c_first);
  if (PASS == kPassQuery) __syncthreads();  // wr
#pragma unroll
  for (int f = 0; f < FPW; ++f)
#pragma unroll
    for (int b = 0; b < R2; ++b) {
      const int t = 16 * (rb2 + b) + r;
      acc[f][b] += lo2[f][b];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[f][b][j] = PASS == kPassQuery ? fmaf(acc[f][b][j], wr[t], zf[f][j] * wr[kChunkTile + t])
                                          : acc[f][b][j] + zf[f][j];
    }

  // ---- + R y
  for (int ct = c_first; ct < c_end; ++ct) {
    const int cols = cols_of(ct);
    __syncthreads();  // P, or the last tile's R and wc, are no longer read
    if (PASS == kPassKey && c_end - c_first > 1) load_wc(ct);
    f32x4 p[2];
    p[0] = zero4();
    p[1] = zero4();
#pragma unroll
    for (int kc = 0; kc < DH / 32; ++kc)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        Frag<T> ub;
        load8(ub, us + (16 * (sr + b) + r) * LDU + 32 * kc + 8 * g);
        mma(p[b], vr[kc], ub);
      }
    if (PASS == kPassKey) __syncthreads();  // wc
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int ci = 16 * sc + 4 * g + j, ri = 16 * (sr + b) + r;
        const float* w = PASS == kPassQuery ? wr + ri : wc + ci;
        p[b][j] = masked(ct, b, j) || ci >= cols ? 0.0f : fmaf(p[b][j], w[0], w[kChunkTile]);
      }
      *reinterpret_cast<f32x4*>(rs + (16 * (sr + b) + r) * LDR + 16 * sc + 4 * g) = p[b];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      Frag<float> ya[FPW];
#pragma unroll
      for (int f = 0; f < FPW; ++f) to_frag(ya[f], y8[ks][f]);
#pragma unroll
      for (int b = 0; b < R2; ++b) {
        Frag<float> pb;
        load8(pb, rs + (16 * (rb2 + b) + r) * LDR + 32 * ks + 8 * g);
#pragma unroll
        for (int f = 0; f < FPW; ++f) mma(acc[f][b], ya[f], pb);
      }
    }
    if (ct + 1 < c_end) load_ry(ct + 1);
  }
  float* dx = a.dx + (head * a.n + t0) * D;
#pragma unroll
  for (int f = 0; f < FPW; ++f)
#pragma unroll
    for (int b = 0; b < R2; ++b) {
      const int t = 16 * (rb2 + b) + r, ft = 16 * (fb + 8 * f) + 4 * g;
      if (t >= rows) continue;
      float* o = dx + (int64_t)t * D + ft;
      if (vec) {
        if (ft < D) store4(o, acc[f][b][0], acc[f][b][1], acc[f][b][2], acc[f][b][3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (ft + j < D) o[j] = acc[f][b][j];
      }
    }
}

template <typename T, int DH, int KB, int PASS>
hipError_t chunk_launch(const ChunkArgs& a, hipStream_t s) {
  using C = CkCfg<T, DH, KB>;
  static_assert(C::lds(true, true) <= (160u << 10), "LDS of a compute unit");
  const hipError_t e = allow_lds<chunk_kernel<T, DH, KB, PASS>>((int)C::lds(true, true));
  if (e != hipSuccess) return e;
  const int64_t tiles = (a.n + kChunkTile - 1) / kChunkTile;
  const int64_t blocks = a.heads * ((tiles - a.first + a.step - 1) / a.step);
  hipLaunchKernelGGL((chunk_kernel<T, DH, KB, PASS>), dim3((unsigned)blocks), dim3(kCkThreads),
                     C::lds(a.causal, PASS == kPassKey || a.u != nullptr), s, a);
  return hipGetLastError();
}
template <typename T, int DH, int PASS>
hipError_t chunk_launch_d(const ChunkArgs& a, hipStream_t s) {
  if (a.D <= 64) return chunk_launch<T, DH, 2, PASS>(a, s);
  if (a.D <= 128) return chunk_launch<T, DH, 4, PASS>(a, s);
  return chunk_launch<T, DH, 8, PASS>(a, s);
}
template <typename T, int PASS>
hipError_t chunk_launch_t(int d, const ChunkArgs& a, hipStream_t s) {
  if (d == 32) return chunk_launch_d<T, 32, PASS>(a, s);
  if (d == 64) return chunk_launch_d<T, 64, PASS>(a, s);
  if (d == 128) return chunk_launch_d<T, 128, PASS>(a, s);
  return hipErrorInvalidValue;
}
template <int PASS>
hipError_t chunk_launch_p(Dt dt, int d, const ChunkArgs& a, hipStream_t s) {
  const int64_t tiles = (a.n + kChunkTile - 1) / kChunkTile;
  return by_heads(a.heads, tiles * kCkThreads, [&](int64_t h0, int64_t hn) {
    const int64_t rows = h0 * a.n, values = rows * d * (dt == Dt::BF16 ? 2 : 4);
    ChunkArgs q = a;
    q.x = a.x + rows * a.D;
    q.y = a.y + rows * a.D;
    q.u = advance(a.u, values);
    q.v = advance(a.v, values);
    q.out = advance(a.out, values);
    q.state = a.state + h0 * a.pieces * a.elems;
    if (a.w) q.w = a.w + rows * 2;
    if (a.dx) q.dx = a.dx + rows * a.D;
    q.heads = hn;
    // An output in the place of the columns (out = V, dV = dO): a tile meets the columns of its
    // piece's tiles up to its own (query pass) or from its own on (key pass), so the tiles of a
    // piece go one after the other, those that the others do not meet first.  dphi(K), for which
    // the key pass reads the columns again, is formed before.
    auto launch = [&]() {
      return dt == Dt::BF16 ? chunk_launch_t<__bf16, PASS>(d, q, s) : chunk_launch_t<float, PASS>(d, q, s);
    };
    q.first = 0;
    q.step = 1;
    if (!a.causal || a.out == nullptr || (a.out != a.v && a.out != (const void*)a.y)) return launch();
    hipError_t e = hipSuccess;
    if (PASS == kPassKey) {
      q.out = nullptr;
      if ((e = launch()) != hipSuccess) return e;
      q.out = advance(a.out, values);
      q.dx = nullptr;
    }
    q.step = a.piece / kChunkTile;
    for (int i = 0; i < q.step && e == hipSuccess; ++i) {
      q.first = PASS == kPassQuery ? q.step - 1 - i : i;
      if (q.first < tiles) e = launch();
    }
    return e;
  });
}

}  // namespace

}  // namespace luna
