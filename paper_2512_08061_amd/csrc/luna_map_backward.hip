// luna_map_backward.hip -- from the gradients of the features back through the feature
// map: dphi -> du -> dx, dW, db and the moments of the channel-MLP gradients.
//
//   map_bwd_kernel  per row: u = W x + b again, the segment of every u, du = sum_l dphi_l
//                   slope_l where the output ReLU passes, dx = W^T du, and per workgroup
//                   the (segment, channel) moments sum dy and sum dy u;
//   map_dw_kernel   [dW | db] = sum over rows of du [x | 1], per workgroup
// (their sums over workgroups, in fp64, are luna_backward.hip's).
//
// Nothing but du (needed again by map_dw_kernel) passes through memory between the
// products: x and dphi are read once, dx written once.
#include <algorithm>

#include "luna_device.hpp"
#include "luna_grad.hpp"
#include "luna_kernels.hpp"
#include "luna_split.hpp"

namespace luna {

namespace {

// an operand, or zeros in the lanes where `keep` is false
__device__ __forceinline__ Frag<float> only(Frag<float> f, bool keep) {
#pragma unroll
  for (int e = 0; e < 8; ++e) f.v[e] = keep ? f.v[e] : 0.0f;
  return f;
}
__device__ __forceinline__ Split3 only(Split3 s, bool keep) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    i32x4 w = __builtin_bit_cast(i32x4, s.p[k].v);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = keep ? w[i] : 0;
    s.p[k].v = __builtin_bit_cast(bf16x8, w);
  }
  return s;
}

// Rows: a parameter set's rows of one side are `segs` runs of `rows` rows, `seg_stride`
// rows apart, the first at row `first` (one run of all heads' rows when the set is
// shared; one run per batch entry otherwise).
struct RowRuns {
  int64_t segs, rows, seg_stride, first;
};
__device__ __forceinline__ RowRuns row_runs(int64_t n, int64_t heads, int H, int per_head, int set) {
  if (!per_head) return RowRuns{1, heads * n, 0, 0};
  return RowRuns{heads / H, n, (int64_t)H * n, (int64_t)set * n};
}

template <int L>
constexpr int wt_blocks() { return (256 / L + 31) / 32; }  // 32-projection blocks of the largest map

// Threads per workgroup: 16 waves where a lane's fragments, dx sums and feature gradients
// nearly fit the 128 registers that leaves it, 8 where they would spill for real (at
// d = 64, L = 8 in bf16, 16 waves spill 16 bytes: the backward call on 768 heads of 197 rows
// with 16 projections takes 464 us, with 32 projections 830; with 8 waves 467 and 841; without
// dx, in the distillation call, the kernel takes 85 and 82.5 us).
template <typename T, int DH, int L, bool PACK>
constexpr int map_threads() {
  constexpr int NT = PACK ? 2 : 1;
  return NT * (DH / 16 * (int)sizeof(T) + DH / 4 + 8) + 10 * L > 112 ? 512 : 1024;
}

// A wave takes TR = 16 rows at a time (row r = lane % 16), computes u^T = W x^T in
// 16-projection blocks, so that a lane holds four projections 16 mb + 4 g + j of its
// row, and looks up and differentiates them in place.  u is summed in fp32 products also
// for bf16 inputs (8 us of a causal call on 2 x 16 heads of 2048 tokens): a u that rounds
// across a kink takes the other side's slope, so a coarser sum shows in dW.  dx^T = W^T du^T takes du from
// the same registers: two projection blocks are one fragment's eight k slots, slot
// (g, e) standing for projection 32 kb + 16 (e / 4) + 4 g + e % 4, and W^T is kept in
// LDS as fragments of that order.
//
// PACK (M <= 8): half the lanes would hold padding projections.  Two tiles of 16 rows
// share the block instead: W fills block rows 0-7 and 8-15, lanes g < 2 keep the first
// tile's projections and g >= 2 the second's, and dx takes du and W^T fragments that are
// zero for the other tile's slots (both: a row that is not finite stays alone).
//
// The moments are LDS atomics in fp64: an fp32 LDS atomic takes 195 cycles per wave
// instruction here (a probe with one workgroup of 8 waves per CU; 3 cycles a lane whatever
// the addresses), an fp64 one 9 to 21.  With fp32 moments they bound this kernel: 170 us
// for 2 x 12 x 32 heads of 512 rows, 8 projections and 8 channels, now 68, of which the
// 200 MB of x, dphi and dx are 41 at the rate of a copy.  With the table they fill most
// of a CU's LDS, so one workgroup runs per CU.
template <typename T, int DH, int L, bool PACK>
__global__ __launch_bounds__((map_threads<T, DH, L, PACK>())) void map_bwd_kernel(MapBwd a) {
  constexpr int NSEG = nseg_cap(L, kFmSegBytes), KS = DH / 32, CB = DH / 16;
  constexpr int NT = PACK ? 2 : 1, TR = 16 * NT;
  constexpr int KB = PACK ? 2 : wt_blocks<L>();
  __shared__ PwlLds<L, NSEG> tab;
  __shared__ double m0[L][NSEG], m1[L][NSEG];
  __shared__ Frag<T> wt[KB][CB][kWave];
  const int set = blockIdx.y, tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int nwaves = blockDim.x / kWave;
  const int g = lane / 16, r = lane % 16;
  const int M = a.M, D = M * L, MB = (M + 15) / 16;
  const T* W = reinterpret_cast<const T*>(a.W) + (size_t)set * M * DH;
  const float* bias = a.b + (size_t)set * M;
  const bool want_dx = a.dxq != nullptr, want_grads = a.duq != nullptr;
  pwl_load(tab, a.tables + (size_t)set * kTableBytes);
  if (want_grads)
    for (int i = tid; i < L * NSEG; i += blockDim.x) {
      (&m0[0][0])[i] = 0.0;
      (&m1[0][0])[i] = 0.0;
    }
  if (want_dx) {
    const int kbs = PACK ? 2 : (MB + 1) / 2;
    for (int i = tid; i < kbs * CB * kWave; i += blockDim.x) {
      const int ln = i % kWave, cb = i / kWave % CB, kb = i / (kWave * CB);
      const int wg = ln / 16, c = 16 * cb + ln % 16;
      Frag<T> f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        int p = 32 * kb + 16 * (e / 4) + 4 * wg + e % 4;
        if constexpr (PACK) p = e < 4 && wg / 2 == kb ? 4 * (wg % 2) + e : M;
        f.set(e, p < M ? (float)W[(size_t)p * DH + c] : 0.0f);
      }
      wt[kb][cb][ln] = f;
    }
  }
  __syncthreads();
  const int steps = __builtin_amdgcn_readfirstlane(tab.steps);
  const float floor = tab.floor;
  const float rsm = 1.0f / sqrtf((float)M);
  const RowRuns rr = row_runs(a.n, a.heads, a.H, a.per_head, set);
  const auto bw = rows_rsrc(W, 0, M, M, DH, sizeof(T));  // (projections past M read as 0)
  const int64_t tps = (rr.rows + TR - 1) / TR, per_side = rr.segs * tps;
  const bool vec = (M * L) % 4 == 0;  // rows of dphi (and, with M % 4, of du) start 16-byte aligned
  const bool vecu = M % 4 == 0;
  // The rows of step t (B operands; past a run's last they read as 0).  With 8 waves, too few
  // to cover their latency, they are asked for a step ahead (92 us instead of 98 for 2 x 65,536
  // rows of 128 elements and 32 projections); 16 waves have no registers for it.
  constexpr bool AHEAD = map_threads<T, DH, L, PACK>() == 512;
  auto load_rows = [&](Frag<T> (&xf)[NT][KS], int64_t t) {
    const bool key = t >= per_side;
    const int64_t ts = key ? t - per_side : t;
    const int64_t seg = rr.segs == 1 ? 0 : ts / tps, t0 = (ts - seg * tps) * TR;
    const auto rs = rows_rsrc(reinterpret_cast<const T*>(key ? a.xk : a.xq) + (rr.first + seg * rr.seg_stride + t0) * DH,
                              0, TR, (int)min((int64_t)TR, rr.rows - t0), DH, sizeof(T));
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        buf_load8(xf[i][ks], rs, ((16 * i + r) * DH + 32 * ks + 8 * g) * (int)sizeof(T));
  };
  const int64_t first = (int64_t)blockIdx.x * nwaves + wave, stride = (int64_t)gridDim.x * nwaves;
  Frag<T> xn[NT][KS];
  if (AHEAD && first < 2 * per_side) load_rows(xn, first);
  for (int64_t t = first; t < 2 * per_side; t += stride) {
    const bool key = t >= per_side;
    const int64_t ts = key ? t - per_side : t;
    const int64_t seg = rr.segs == 1 ? 0 : ts / tps, t0 = (ts - seg * tps) * TR;
    const int64_t base = rr.first + seg * rr.seg_stride;
    const float* dphi = key ? a.dphik : a.dphiq;
    // this lane's row of each tile, and the row whose projections it holds
    int64_t xrow[NT];
    bool xok[NT];
    Frag<T> xf[NT][KS];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int64_t tr = t0 + 16 * i + r;
      xok[i] = tr < rr.rows;
      xrow[i] = base + (xok[i] ? tr : t0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if constexpr (AHEAD) xf[i][ks] = xn[i][ks];
    }
    if constexpr (!AHEAD) load_rows(xf, t);
    else if (t + stride < 2 * per_side) load_rows(xn, t + stride);
    const int mine = PACK ? g / 2 : 0;  // the tile whose projections this lane holds
    const int64_t row = mine ? xrow[NT - 1] : xrow[0];
    const bool ok = mine ? xok[NT - 1] : xok[0];
    const int pg = PACK ? 4 * (g % 2) : 4 * g;  // its first projection within a block
    f32x4 dx[NT][CB];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) dx[i][cb] = zero4();
    float du[8];
    for (int mb = 0; mb < MB; ++mb) {
      const int p0 = 16 * mb + pg;
      float gv[4][L];
      if (vec && ok && p0 + 3 < M) {
        const float4* gp = reinterpret_cast<const float4*>(dphi + row * D + (int64_t)p0 * L);
#pragma unroll
        for (int q = 0; q < L; ++q) reinterpret_cast<float4*>(&gv[0][0])[q] = gp[q];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int l = 0; l < L; ++l)
            gv[j][l] = ok && p0 + j < M ? dphi[row * D + (int64_t)(p0 + j) * L + l] : 0.0f;
      }
      f32x4 us[NT];
#pragma unroll
      for (int i = 0; i < NT; ++i) us[i] = zero4();
      const int prow = PACK ? r % 8 : 16 * mb + r;  // W row this lane feeds to the A operand
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        Frag<T> wf;
        buf_load8(wf, bw, (prow * DH + 32 * ks + 8 * g) * (int)sizeof(T));
#pragma unroll
        for (int i = 0; i < NT; ++i) mma(us[i], widen(wf), widen(xf[i][ks]));
      }
      const f32x4 acc = mine ? us[NT - 1] : us[0];
      float u[4];
      int sg[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = acc[j] + (p0 + j < M ? bias[p0 + j] : 0.0f);
      pwl_search(tab, steps, u, sg);
      float d4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float2* srow = reinterpret_cast<const float2*>(seg_ptr(tab, sg[j]));
        float s = 0.0f, dy[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
          const float2 st = srow[l];
          const float gl = fmaf(st.x, u[j], st.y) > floor ? gv[j][l] : 0.0f;  // floor: 0 (output ReLU) or -inf
          s = fmaf(gl, st.x, s);
          dy[l] = gl * rsm;
        }
        if (want_grads)
#pragma unroll
          for (int l = 0; l < L; ++l)
            if (dy[l] != 0.0f) {  // (channels cut by the output ReLU, and padding, add nothing)
              atomicAdd(&m0[l][sg[j]], (double)dy[l]);
              atomicAdd(&m1[l][sg[j]], (double)(dy[l] * u[j]));
            }
        d4[j] = s;
      }
      if (want_grads && ok) {
        float* dst = (key ? a.duk : a.duq) + row * M + p0;
        if (vecu && p0 + 3 < M) {
          store4(dst, d4[0], d4[1], d4[2], d4[3]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (p0 + j < M) dst[j] = d4[j];
        }
      }
      if (!want_dx) continue;
      const int half = PACK ? 0 : mb % 2;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (half == 0) {
          du[j] = d4[j];
          du[4 + j] = 0.0f;
        } else {
          du[4 + j] = d4[j];
        }
      }
      if (half == 0 && mb + 1 < MB) continue;  // (uniform) the next block fills the other half
      Frag<float> df;
#pragma unroll
      for (int e = 0; e < 8; ++e) df.v[e] = du[e];
      Operand<float, T> dw;
      set_operand(dw, df);
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        // (the other tile's slots as 0: W^T's own zeros would turn its infinities into NaN here)
        const Operand<float, T> di = PACK ? only(dw, mine == i) : dw;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) mma(dx[i][cb], wt[PACK ? i : mb / 2][cb][lane], di);
      }
    }
    if (!want_dx) continue;
    T* dX = reinterpret_cast<T*>(key ? a.dxk : a.dxq);
#pragma unroll
    for (int i = 0; i < NT; ++i)
      if (xok[i])
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          store4(dX + xrow[i] * DH + 16 * cb + 4 * g, dx[i][cb][0], dx[i][cb][1], dx[i][cb][2], dx[i][cb][3]);
  }
  if (!want_grads) return;
  __syncthreads();
  float2* part = reinterpret_cast<float2*>(a.partial + ((size_t)set * gridDim.x + blockIdx.x) * a.part_floats);
  const int nm = tab.zero_seg * L;  // real segments x channels
  for (int i = tid; i < nm; i += blockDim.x) {  // partials as [segment][channel][2]
    part[i] = make_float2((float)m0[i % L][i / L], (float)m1[i % L][i / L]);
  }
}

// ---------------------------------------------------------------------------
// [dW | db] of 32 projections over a workgroup's rows.  A wave takes 32 rows at a time
// as the k dimension of one fragment: du^T straight from memory (16 lanes read 64
// consecutive bytes of a row), x transposed through its own LDS tile.  Bound by the
// reads of du and x.
// ---------------------------------------------------------------------------
constexpr int kDwRows = 32, kDwProj = 32;

template <typename T, int DH>
__global__ __launch_bounds__(256) void map_dw_kernel(MapBwd a) {
  constexpr int CB = DH / 16, LD = DH + 16 / (int)sizeof(T), V = Vec16<T>::N;
  constexpr size_t kTile = (size_t)kDwRows * LD * sizeof(T), kOut = (size_t)kDwProj * (DH + 1) * 4;
  __shared__ __attribute__((aligned(16))) char lds[4 * (kTile > kOut ? kTile : kOut)];
  const int set = blockIdx.z, pb = blockIdx.y * kDwProj;
  const int tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int g = lane / 16, r = lane % 16;
  const int M = a.M;
  T* xs = reinterpret_cast<T*>(lds + wave * kTile);
  f32x4 acc[2][CB];
  float db[2] = {0.0f, 0.0f};
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[x][cb] = zero4();
  const RowRuns rr = row_runs(a.n, a.heads, a.H, a.per_head, set);
  const int64_t tps = (rr.rows + kDwRows - 1) / kDwRows, per_side = rr.segs * tps;
  for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < 2 * per_side; t += (int64_t)gridDim.x * 4) {
    const bool key = t >= per_side;
    const int64_t ts = key ? t - per_side : t;
    const int64_t seg = ts / tps, t0 = (ts - seg * tps) * kDwRows;
    const int64_t base = rr.first + seg * rr.seg_stride + t0;
    const int rows = (int)min((int64_t)kDwRows, rr.rows - t0);
    const T* X = reinterpret_cast<const T*>(key ? a.xk : a.xq) + base * DH;
    const float* du = (key ? a.duk : a.duq) + base * M;
    Frag<float> v[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int p = pb + 16 * x + r, k = 8 * g + e;
        v[x].v[e] = p < M && k < rows ? du[(int64_t)k * M + p] : 0.0f;
      }
    // the tile's x rows (zero past the last, so that padding rows add 0)
    constexpr int PER = kDwRows * DH / V / kWave;
    uint4 xv[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = lane + i * kWave, k = c / (DH / V), q = c % (DH / V);
      xv[i] = k < rows ? reinterpret_cast<const uint4*>(X + (int64_t)k * DH)[q] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = lane + i * kWave, k = c / (DH / V), q = c % (DH / V);
      *reinterpret_cast<uint4*>(xs + k * LD + q * V) = xv[i];
    }
    wave_lds_fence();
    Operand<float, T> w[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      set_operand(w[x], v[x]);
#pragma unroll
      for (int e = 0; e < 8; ++e) db[x] += v[x].v[e];
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      Frag<T> xf;
      load_tr4(xf, 0, xs, LD, 8 * g, 16 * cb, lane);
      load_tr4(xf, 4, xs, LD, 8 * g + 4, 16 * cb, lane);
#pragma unroll
      for (int x = 0; x < 2; ++x)
        if (pb + 16 * x < M) mma(acc[x][cb], w[x], xf);  // (uniform)
    }
    wave_lds_fence();
  }
  // db: the four lane groups hold different rows of projection r
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    db[x] += __shfl_xor(db[x], 16, kWave);
    db[x] += __shfl_xor(db[x], 32, kWave);
  }
  __syncthreads();
  float* out = reinterpret_cast<float*>(lds);  // [wave][projection][DH + 1]
  float* mine = out + wave * kDwProj * (DH + 1);
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 4; ++j) mine[(16 * x + 4 * g + j) * (DH + 1) + 16 * cb + r] = acc[x][cb][j];
    if (g == 0) mine[(16 * x + r) * (DH + 1) + DH] = db[x];
  }
  __syncthreads();
  const int np = min(kDwProj, M - pb);
  float* dst = a.dw_partial + (((size_t)set * gridDim.x + blockIdx.x) * M + pb) * (DH + 1);
  for (int i = tid; i < np * (DH + 1); i += blockDim.x) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += out[w * kDwProj * (DH + 1) + i];
    dst[i] = s;
  }
}

template <typename T, int DH, int L>
hipError_t map_launch_L(const MapBwd& a, int sets, hipStream_t s) {
  const dim3 grid((unsigned)a.groups, (unsigned)sets);
  // (fp32, d = 128, L = 16: the table, the moments and two sets of W^T fragments exceed LDS)
  constexpr bool can_pack = !(sizeof(T) == 4 && DH == 128 && L == 16);
  if constexpr (can_pack)
    if (a.M <= 8) {
      hipLaunchKernelGGL((map_bwd_kernel<T, DH, L, true>), grid, dim3(map_threads<T, DH, L, true>()), 0, s, a);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((map_bwd_kernel<T, DH, L, false>), grid, dim3(map_threads<T, DH, L, false>()), 0, s, a);
  return hipGetLastError();
}

template <typename T, int DH>
hipError_t map_launch_d(int L, const MapBwd& a, int sets, hipStream_t s) {
  auto launch = [&](const MapBwd& q) {
    switch (L) {
      case 1: return map_launch_L<T, DH, 1>(q, sets, s);
      case 2: return map_launch_L<T, DH, 2>(q, sets, s);
      case 4: return map_launch_L<T, DH, 4>(q, sets, s);
      case 8: return map_launch_L<T, DH, 8>(q, sets, s);
      case 16: return map_launch_L<T, DH, 16>(q, sets, s);
      default: return hipErrorInvalidValue;
    }
  };
  // dx in the place of x: after map_dw_kernel, which reads x too
  const bool late = a.duq && a.dxq && (a.dxq == a.xq || a.dxk == a.xk);
  MapBwd q = a;
  if (late) q.dxq = q.dxk = nullptr;
  hipError_t e = launch(q);
  if (e != hipSuccess || a.duq == nullptr) return e;
  const dim3 grid((unsigned)a.dw_groups, (unsigned)((a.M + kDwProj - 1) / kDwProj), (unsigned)sets);
  hipLaunchKernelGGL((map_dw_kernel<T, DH>), grid, dim3(256), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess || !late) return e;
  q = a;
  q.duq = q.duk = nullptr;
  return launch(q);
}

template <typename T>
hipError_t map_launch(int d, int L, const MapBwd& a, int sets, hipStream_t s) {
  switch (d) {
    case 32: return map_launch_d<T, 32>(L, a, sets, s);
    case 64: return map_launch_d<T, 64>(L, a, sets, s);
    case 128: return map_launch_d<T, 128>(L, a, sets, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Workgroups per parameter set: one per CU over all sets (each fills a CU's LDS), fewer
// when the 16-row tiles of both sides are fewer than their waves.
int map_bwd_groups(int64_t rows_per_set, int sets) {
  const int64_t want = (256 + sets - 1) / sets, most = (2 * rows_per_set + 255) / 256;
  return (int)std::max<int64_t>(1, std::min(want, most));
}
// Workgroups of the weight-gradient products: two per CU over all sets, at least eight
// 32-row tiles per wave (fewer partials to sum).
int map_dw_groups(int64_t rows_per_set, int sets) {
  const int64_t want = (512 + sets - 1) / sets, most = (2 * rows_per_set + 1023) / 1024;
  return (int)std::max<int64_t>(1, std::min(want, most));
}

hipError_t launch_map_bwd(Dt dt, int d, int L, const MapBwd& a, int sets, hipStream_t s) {
  return dt == Dt::BF16 ? map_launch<__bf16>(d, L, a, sets, s) : map_launch<float>(d, L, a, sets, s);
}

}  // namespace luna
