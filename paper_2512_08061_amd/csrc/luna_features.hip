// luna_features.hip -- kernel attention, eq. (9) of Section 3.1, from features in memory:
//
//   feat_state_kernel    S = phi(K)^T V and z = phi(K)^T 1 per piece of a head's tokens
//   feat_total_kernel    the pieces of a head summed
//   feat_readout_kernel  out = phi(Q) S / (phi(Q) z + eps)
//   feat_export_kernel   the statistics in the caller's layout
//
// The sums are fp32 whatever the types: two bf16 operands multiply exactly, a bf16 and
// an fp32 one as three bf16 products, two fp32 ones on the fp32 matrix cores.  Features
// and values are read in their own types, and z and the denominators are formed beside
// the products, so nothing is widened or packed in memory first.  (Widening the features,
// packing [V | 1], fp32 products on padded tiles and a scan took 440 us for 64 heads of
// 4096 tokens with 128 bf16 features and d = 64; these kernels take 20 + 5 + 30 us.)
#include <algorithm>

#include "luna_device.hpp"
#include "luna_features.hpp"
#include "luna_split.hpp"

namespace luna {

namespace {

// Features, values and statistics are read through range-checked buffers that end with their
// last row, so that rows past it read as 0: a test per load puts a branch around each.
__device__ __forceinline__ uint4 piece16(Buf b, int off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}

// ---------------------------------------------------------------------------
// Per piece: S = phi(K)^T V, z.  Workgroups of four waves stage 32 tokens of features
// and values in LDS (the next 32 in registers meanwhile) and read both transposed, the
// tokens being the k dimension; wave w forms the 16-feature blocks w, w + 4, ... and all
// value columns.  Bound by the read of the features and values: pieces are short enough
// that a few hundred workgroups share the device; where they are few all the same, a step is
// bound by its products (4.9 us for 256 fp32 features beside d = 128), and a piece's features
// go to two or four workgroups that each read its values (a call on 1 head of 512 tokens 38 ->
// 28 us).
// ---------------------------------------------------------------------------
constexpr int kFsTok = 32;

template <typename TF, typename T, int DH, int FBW, bool WGT>
__global__ __launch_bounds__(256) void feat_state_kernel(FeatArgs a) {
  constexpr int CB = DH / 16, VF = Vec16<TF>::N, VT = Vec16<T>::N;
  constexpr int DPM = 64 * FBW;                                  // features at most
  constexpr int LDP = DPM + 16 / (int)sizeof(TF), LDV = DH + 16 / (int)sizeof(T);
  constexpr int NP = kFsTok * DPM / VF / 256, NV = (kFsTok * DH / VT + 255) / 256;
  __shared__ __attribute__((aligned(16))) TF ps[kFsTok * LDP];
  __shared__ __attribute__((aligned(16))) T vs[kFsTok * LDV];
  __shared__ float2 ws[WGT ? kFsTok : 1];
  const int64_t head = blockIdx.x / a.pieces;
  const int piece = (int)(blockIdx.x - head * a.pieces);
  const int64_t first = (int64_t)piece * a.piece;
  const int rows = (int)min((int64_t)a.piece, a.n - first);
  const int D = a.D, tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int g = lane / 16, r = lane % 16;
  const int from = blockIdx.y * DPM;  // this workgroup's first feature
  const TF* phi = reinterpret_cast<const TF*>(a.phik) + (head * a.n + first) * D;
  const T* V = reinterpret_cast<const T*>(a.v) + (head * a.n + first) * DH;
  const bool vec = D % VF == 0;  // (uniform) feature rows are whole 16-byte pieces
  f32x4 acc[FBW][CB];
  float z[FBW];
#pragma unroll
  for (int f = 0; f < FBW; ++f) {
    z[f] = 0.0f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[f][cb] = zero4();
  }
  uint4 pr[NP], vr[NV];
  const Buf bphi = buffer(phi, rows * D * (int)sizeof(TF)), bv = buffer(V, rows * DH * (int)sizeof(T));
  auto load = [&](int t0) {
    if (vec)
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int c = tid + 256 * i, q = from + c % (DPM / VF) * VF;
        pr[i] = piece16(bphi, q < D ? ((t0 + c / (DPM / VF)) * D + q) * (int)sizeof(TF) : kPastEnd);
      }
#pragma unroll
    for (int i = 0; i < NV; ++i) vr[i] = piece16(bv, t0 * DH * (int)sizeof(T) + (tid + 256 * i) * 16);
  };
  load(0);
  for (int t0 = 0; t0 < rows; t0 += kFsTok) {
    if (t0) __syncthreads();  // every wave is done with the tile
    if (vec) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int c = tid + 256 * i;
        *reinterpret_cast<uint4*>(ps + c / (DPM / VF) * LDP + c % (DPM / VF) * VF) = pr[i];
      }
    } else {
      for (int i = tid; i < kFsTok * DPM; i += 256) {
        const int k = i / DPM, f = from + i % DPM;
        ps[k * LDP + i % DPM] = t0 + k < rows && f < D ? phi[(int64_t)(t0 + k) * D + f] : (TF)0.0f;
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = tid + 256 * i;
      if (c < kFsTok * DH / VT) *reinterpret_cast<uint4*>(vs + c / (DH / VT) * LDV + c % (DH / VT) * VT) = vr[i];
    }
    if (WGT && tid < kFsTok)
      ws[tid] = t0 + tid < rows ? reinterpret_cast<const float2*>(a.w)[head * a.n + first + t0 + tid]
                                : make_float2(0.0f, 0.0f);
    __syncthreads();
    if (t0 + kFsTok < rows) load(t0 + kFsTok);
    Operand<TF, T> af[FBW];
#pragma unroll
    for (int f = 0; f < FBW; ++f) {
      const int fb = wave + 4 * f;
      Frag<TF> x;
      load_tr4(x, 0, ps, LDP, 8 * g, 16 * fb, lane);
      load_tr4(x, 4, ps, LDP, 8 * g + 4, 16 * fb, lane);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (WGT) {
          const float2 w = ws[8 * g + e];
          z[f] = fmaf(x.v[e], w.y, z[f]);
          x.v[e] *= w.x;
        } else {
          z[f] += x.get(e);
        }
      }
      if constexpr (sizeof(TF) > sizeof(T)) split3<false>(af[f], x.v);  // (checked below)
      else set_operand(af[f], x);
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      Frag<T> y;
      load_tr4(y, 0, vs, LDV, 8 * g, 16 * cb, lane);
      load_tr4(y, 4, vs, LDV, 8 * g + 4, 16 * cb, lane);
      Operand<T, TF> bf;
      set_operand(bf, y);
#pragma unroll
      for (int f = 0; f < FBW; ++f)
        if (f == 0 || from + 16 * (wave + 4 * f) < D) mma(acc[f][cb], af[f], bf);  // (uniform)
    }
  }
  float* S = a.state + blockIdx.x * a.elems;
  auto store = [&](const f32x4& c, int f, int cb) {
    const int f0 = from + 16 * (wave + 4 * f) + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (f0 + j < D) S[(f0 + j) * DH + 16 * cb + r] = c[j];
  };
  float nan = 0.0f;  // until a sum is NaN (or infinite)
#pragma unroll
  for (int f = 0; f < FBW; ++f) {
    z[f] += __shfl_xor(z[f], 16, kWave);
    z[f] += __shfl_xor(z[f], 32, kWave);
    const int f0 = from + 16 * (wave + 4 * f);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const f32x4 c = acc[f][cb];
      store(c, f, cb);
      nan = fmaf(c[0] + c[1], 0.0f, fmaf(c[2] + c[3], 0.0f, nan));
    }
    if (g == 0 && f0 + r < D) S[D * DH + f0 + r] = z[f];
  }
  // fp32 features beside bf16 values: an infinite value, or a feature above the largest bf16
  // one, has met parts of either sign, and such sums end as NaN.  They are formed again as fp32
  // products, each wave's from memory.
  if constexpr (sizeof(TF) > sizeof(T))
    if (__any(nan != 0.0f)) {  // (uniform)
#pragma unroll 1
      for (int cb = 0; cb < CB; ++cb) {
        f32x4 c[FBW];
#pragma unroll
        for (int f = 0; f < FBW; ++f) c[f] = zero4();
        for (int t0 = 0; t0 < rows; t0 += kFsTok) {
          Frag<float> x[FBW];
          Frag<T> y;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int t = t0 + 8 * g + e;
            const float w = WGT && t < rows ? reinterpret_cast<const float2*>(a.w)[head * a.n + first + t].x : 1.0f;
#pragma unroll
            for (int f = 0; f < FBW; ++f) {
              const int k = from + 16 * (wave + 4 * f) + r;
              x[f].v[e] = w * __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                  bphi, k < D ? (t * D + k) * (int)sizeof(TF) : kPastEnd, 0, 0));
            }
            y.v[e] = __builtin_bit_cast(
                T, __builtin_amdgcn_raw_buffer_load_b16(bv, (t * DH + 16 * cb + r) * (int)sizeof(T), 0, 0));
          }
#pragma unroll
          for (int f = 0; f < FBW; ++f) mma(c[f], x[f], widen(y));
        }
#pragma unroll
        for (int f = 0; f < FBW; ++f) store(c[f], f, cb);
      }
    }
}

// ---------------------------------------------------------------------------
// the pieces of every head summed into its first, in order
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void feat_total_kernel(float* state, int64_t heads, int pieces, int64_t elems) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= heads * elems) return;
  const int64_t h = i / elems, e = i - h * elems;
  float* p = state + h * pieces * elems + e;
  float s = 0.0f;
  int c = 0;
  for (; c + 8 <= pieces; c += 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[(c + k) * elems];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  if (c + 4 <= pieces) {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = p[(c + k) * elems];
#pragma unroll
    for (int k = 0; k < 4; ++k) s += v[k];
    c += 4;
  }
  for (; c < pieces; ++c) s += p[c * elems];
  *p = s;
}

// ---------------------------------------------------------------------------
// Readout, transposed: [num | den]^T = [S | z]^T phi(Q)^T, so that a lane reads 8
// consecutive features of one query straight into a B operand and ends with 4
// consecutive outputs of it.  [S | z]^T waits in LDS as A fragments (z as one block of 16
// equal rows: every lane then holds its query's den), up to four value blocks per
// workgroup; a fragment read serves NTL tiles of 16 queries.  Bound by the read of phi(Q).
// ---------------------------------------------------------------------------
constexpr int kFrThreads = 512;

template <typename TF>
constexpr int readout_tiles() { return sizeof(TF) == 2 ? 2 : 1; }

template <typename TF, typename T, int DH, int KB>
__global__ __launch_bounds__(kFrThreads) void feat_readout_kernel(FeatArgs a) {
  constexpr int CB = DH / 16, CBW = CB < 4 ? CB : 4, NTL = readout_tiles<TF>();
  using AOp = Operand<float, TF>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  AOp* frags = reinterpret_cast<AOp*>(lds);  // [kb][CBW + 1][lane]
  const int64_t per_head = (a.n + a.tokens - 1) / a.tokens;
  const int64_t head = blockIdx.x / per_head;
  const int64_t first = (blockIdx.x - head * per_head) * a.tokens;
  const int64_t last = min(a.n, first + a.tokens);
  const int c0 = blockIdx.y * CBW * 16;
  const int D = a.D, tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int g = lane / 16, r = lane % 16;
  const int kbs = (D + 31) / 32;
  const Buf bS = buffer(a.state + head * a.pieces * a.elems, D * (DH + 1) * 4);
  // (every load of a thread's fragments before the first is split: in turn, the five rounds
  // of 256 features took 20 us of a short call)
  constexpr int NI = (KB * (CBW + 1) * kWave + kFrThreads - 1) / kFrThreads;
  Frag<float> fr[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int at = tid + kFrThreads * i, ln = at % kWave, blk = at / kWave % (CBW + 1), kb = at / (kWave * (CBW + 1));
    const int k0 = 32 * kb + 8 * (ln / 16), c = c0 + 16 * blk + ln % 16;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = k0 + e, el = blk < CBW ? k * DH + c : D * DH + k;
      fr[i].v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(bS, k < D ? 4 * el : kPastEnd, 0, 0));
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
    if (tid + kFrThreads * i < kbs * (CBW + 1) * kWave) set_operand(frags[tid + kFrThreads * i], fr[i]);
  __syncthreads();
  const TF* phi = reinterpret_cast<const TF*>(a.phiq) + (head * a.n + first) * D;
  T* out = reinterpret_cast<T*>(a.out) + head * a.n * DH;
  const bool vec = D % Vec16<TF>::N == 0 && D % 8 == 0;  // (uniform)
  for (int64_t t0 = first + wave * 16 * NTL; t0 < last; t0 += (kFrThreads / kWave) * 16 * NTL) {
    Frag<TF> q[NTL][KB];
#pragma unroll
    for (int i = 0; i < NTL; ++i) {
      const int t = (int)(t0 - first) + 16 * i + r;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int k0 = 32 * kb + 8 * g;
        q[i][kb].zero();
        if (vec) {
          if (first + t < last && k0 < D) load8(q[i][kb], phi + t * D + k0);
        } else if (first + t < last) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (k0 + e < D) q[i][kb].v[e] = phi[t * D + k0 + e];
        }
      }
    }
    f32x4 acc[NTL][CBW + 1];
#pragma unroll
    for (int i = 0; i < NTL; ++i)
#pragma unroll
      for (int b = 0; b <= CBW; ++b) acc[i][b] = zero4();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (kb > 0 && kb >= kbs) break;  // (uniform)
#pragma unroll
      for (int b = 0; b <= CBW; ++b) {
        const AOp& f = frags[(kb * (CBW + 1) + b) * kWave + lane];
#pragma unroll
        for (int i = 0; i < NTL; ++i) mma(acc[i][b], f, q[i][kb]);
      }
    }
#pragma unroll
    for (int i = 0; i < NTL; ++i) {
      const int64_t t = t0 + 16 * i + r;
      if (t >= last) continue;
      const float inv = 1.0f / (acc[i][CBW][0] + a.eps);
      T* o = out + t * DH + c0 + 4 * g;
#pragma unroll
      for (int b = 0; b < CBW; ++b)
        store4(o + 16 * b, acc[i][b][0] * inv, acc[i][b][1] * inv, acc[i][b][2] * inv, acc[i][b][3] * inv);
    }
  }
}

// ---------------------------------------------------------------------------
// statistics into (or added to) the caller's S and z
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void feat_export_kernel(const float* __restrict__ state, int64_t head_stride,
                                                          float* __restrict__ S, float* __restrict__ z, int64_t heads,
                                                          int D, int d, int accumulate) {
  const int64_t per = (int64_t)D * (d + 1);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < heads * per;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t h = i / per, e = i - h * per;
    const float v = state[h * head_stride + e];
    float* dst = e < (int64_t)D * d ? S + h * D * d + e : z + h * D + (e - (int64_t)D * d);
    *dst = accumulate ? *dst + v : v;
  }
}

template <typename TF, typename T, int DH, bool WGT>
hipError_t state_launch_w(const FeatArgs& a, hipStream_t s) {
  const int each = feat_state_features(a.D, a.heads * a.pieces);
  const dim3 grid((unsigned)(a.heads * a.pieces), (unsigned)((a.D + each - 1) / each)), block(256);
  if (each == 64) hipLaunchKernelGGL((feat_state_kernel<TF, T, DH, 1, WGT>), grid, block, 0, s, a);
  else if (each == 128) hipLaunchKernelGGL((feat_state_kernel<TF, T, DH, 2, WGT>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((feat_state_kernel<TF, T, DH, 4, WGT>), grid, block, 0, s, a);
  return hipGetLastError();
}
template <typename TF, typename T, int DH>
hipError_t state_launch(const FeatArgs& a, hipStream_t s) {
  if (a.w == nullptr) return state_launch_w<TF, T, DH, false>(a, s);
  if constexpr (sizeof(TF) == 4) return state_launch_w<TF, T, DH, true>(a, s);
  return hipErrorInvalidValue;  // (weights go with fp32 features)
}

template <auto Kernel>
hipError_t readout_launch_k(dim3 grid, size_t lds, const FeatArgs& a, hipStream_t s) {
  if (lds > (64u << 10)) {
    const hipError_t e = allow_lds<Kernel>(160 << 10);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(Kernel, grid, dim3(kFrThreads), lds, s, a);
  return hipGetLastError();
}

template <typename TF, typename T, int DH>
hipError_t readout_launch(const FeatArgs& args, hipStream_t s) {
  constexpr int CB = DH / 16, CBW = CB < 4 ? CB : 4;
  FeatArgs a = args;
  // one pass of a workgroup's waves over its tokens; more passes, up to 1024 tokens, as long as
  // about two workgroups per CU remain (the fragments are set up once per workgroup)
  constexpr int kPass = kFrThreads / kWave * 16 * readout_tiles<TF>();
  const int64_t passes = a.heads * a.n / (512 * kPass);
  a.tokens = kPass * (int)std::max<int64_t>(1, std::min<int64_t>(1024 / kPass, passes));
  const int64_t blocks = a.heads * ((a.n + a.tokens - 1) / a.tokens);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, (unsigned)(CB / CBW));
  const size_t lds = (size_t)((a.D + 31) / 32) * (CBW + 1) * kWave * sizeof(Operand<float, TF>);
  if (a.D <= 64) return readout_launch_k<feat_readout_kernel<TF, T, DH, 2>>(grid, lds, a, s);
  if (a.D <= 128) return readout_launch_k<feat_readout_kernel<TF, T, DH, 4>>(grid, lds, a, s);
  return readout_launch_k<feat_readout_kernel<TF, T, DH, 8>>(grid, lds, a, s);
}

// f(type tags) for the feature and value types, F::operator()<TF, T, DH>
template <typename F>
hipError_t by_type(Dt fdt, Dt vdt, int d, F f) {
  auto by_d = [&](auto tf, auto t) {
    using TF = decltype(tf);
    using T = decltype(t);
    switch (d) {
      case 32: return f.template operator()<TF, T, 32>();
      case 64: return f.template operator()<TF, T, 64>();
      case 128: return f.template operator()<TF, T, 128>();
      default: return hipErrorInvalidValue;
    }
  };
  if (fdt == Dt::BF16) return vdt == Dt::BF16 ? by_d(__bf16(), __bf16()) : by_d(__bf16(), float());
  return vdt == Dt::BF16 ? by_d(float(), __bf16()) : by_d(float(), float());
}

struct StateLaunch {
  const FeatArgs& a;
  hipStream_t s;
  template <typename TF, typename T, int DH>
  hipError_t operator()() const { return state_launch<TF, T, DH>(a, s); }
};
struct ReadoutLaunch {
  const FeatArgs& a;
  hipStream_t s;
  template <typename TF, typename T, int DH>
  hipError_t operator()() const { return readout_launch<TF, T, DH>(a, s); }
};

}  // namespace

// Value widths of whole fragments, and feature counts up to four 16-feature blocks a wave.
bool feat_supported(int d, int D) { return (d == 32 || d == 64 || d == 128) && D >= 1 && D <= 256; }

// the arguments of heads h0 .. h0 + hn - 1
static FeatArgs feat_heads(const FeatArgs& a, Dt fdt, Dt vdt, int d, int64_t h0, int64_t hn) {
  const int64_t rows = h0 * a.n, fs = fdt == Dt::BF16 ? 2 : 4, vs = vdt == Dt::BF16 ? 2 : 4;
  FeatArgs q = a;
  q.phiq = advance(a.phiq, rows * a.D * fs);
  q.phik = advance(a.phik, rows * a.D * fs);
  q.v = advance(a.v, rows * d * vs);
  q.out = advance(a.out, rows * d * vs);
  q.state = a.state + h0 * a.pieces * a.elems;
  if (a.w) q.w = a.w + rows * 2;
  q.heads = hn;
  return q;
}

hipError_t launch_feat_state(Dt fdt, Dt vdt, int d, const FeatArgs& a, hipStream_t s) {
  return by_heads(a.heads, (int64_t)a.pieces * 256, [&](int64_t h0, int64_t hn) {
    const FeatArgs q = feat_heads(a, fdt, vdt, d, h0, hn);
    return by_type(fdt, vdt, d, StateLaunch{q, s});
  });
}

hipError_t launch_feat_total(const FeatArgs& a, hipStream_t s) {
  if (a.pieces == 1) return hipSuccess;
  return by_heads(a.heads, a.elems + 256, [&](int64_t h0, int64_t hn) {
    hipLaunchKernelGGL(feat_total_kernel, dim3((unsigned)((hn * a.elems + 255) / 256)), dim3(256), 0, s,
                       a.state + h0 * a.pieces * a.elems, hn, a.pieces, a.elems);
    return hipGetLastError();
  });
}

hipError_t launch_feat_readout(Dt fdt, Dt vdt, int d, const FeatArgs& a, hipStream_t s) {
  return by_heads(a.heads, (a.n + 127) / 128 * kFrThreads * 2, [&](int64_t h0, int64_t hn) {
    const FeatArgs q = feat_heads(a, fdt, vdt, d, h0, hn);
    return by_type(fdt, vdt, d, ReadoutLaunch{q, s});
  });
}

hipError_t launch_feat_export(int d, const FeatArgs& a, float* S, float* z, int accumulate, hipStream_t s) {
  const int64_t elems = (int64_t)a.D * (d + 1);
  const dim3 grid((unsigned)std::min<int64_t>((a.heads * elems + 255) / 256, 65536));
  hipLaunchKernelGGL(feat_export_kernel, grid, dim3(256), 0, s, a.state, a.pieces * a.elems, S, z, a.heads, a.D, d,
                     accumulate);
  return hipGetLastError();
}

}  // namespace luna
