// luna_backward.hip -- gradients of LUNA attention (training the feature map end to
// end and fine-tuning converted models).
//
// For a loss L with upstream gradient dO = dL/dout, with num = phi(Q) S, den = phi(Q) z
// + eps and out = num / den per row (eq. (9) of Section 3.1; prefix states for the
// causal form), the chain rule gives, per row t and with G_t = [dnum_t | dden_t],
//   dnum_t = dO_t / den_t,  dden_t = -(dO_t . num_t) / den_t^2,
//   dphi(q_t) = G_t [S_t | z_t]^T,
//   [dS | dz] = phi(Q)^T G  (non-causal; causal: suffix sums over t >= s),
//   dphi(k_s) = [v_s | 1] [dS_s | dz_s]^T,  dv_s = dS_s^T phi(k_s),
// and through the feature map phi_{iL+l} = relu(y_l(u_i)) / sqrt(M), u = x W^T + b,
// y_l(u) = g_l + sum_k f_lk relu(a_lk u + c_lk) (ReLU'(0) = 0).
//
// The causal form is taken in chunks of C tokens: with the exclusive prefix state
// [S_c | z_c] before chunk c and P_c = tril(phi(Q_c) phi(K_c)^T),
//   [num | den - eps]_c = phi(Q_c) [S_c | z_c] + P_c [V_c | 1],
//   dphi(Q_c) = G_c [S_c | z_c]^T + R_c phi(K_c),   R_c = tril(G_c [V_c | 1]^T),
// and with the exclusive suffix state [dS_c | dz_c] after chunk c,
//   dphi(K_c) = [V_c | 1] [dS_c | dz_c]^T + R_c^T phi(Q_c),
//   dV_c = phi(K_c) dS_c + P_c^T dnum_c,
// an exact regrouping of the sums.  The non-causal form is the same with the total
// state in place of the prefix and suffix states and no intra-chunk terms (its
// chunks only split the sums over tokens among more workgroups).
//
// The attention part runs in luna_features.hip (states of pieces of the tokens) and
// luna_chunk_kernel.hpp (scans, dphi and dV), the feature map's in luna_map_backward.hip
// (dphi -> du -> dx, [dW | db] per workgroup and the (segment, channel) moments sum dy and
// sum dy u of the channel outputs' gradients).  Here:
//   bwd_dw_kernel       [dW | db] summed over workgroups (fp64);
//   bwd_reduce_kernel   the partials summed over workgroups (fp64);
//   bwd_prefix_kernel   exclusive prefix sums of the moments over segments, per channel;
//   bwd_mlp_kernel      the channel-MLP parameter gradients from the moments: unit k
//                       is on exactly on the segments above (a_k > 0) or below
//                       (a_k < 0) its breakpoint, where h_k = a_k u + c_k, so
//                       dfc2_lk = a_k sum_on dy_l u + c_k sum_on dy_l,
//                       dfc1_(l)k = f_lk sum_on dy_l u, dfc1_b likewise, dfc2_b_l = sum dy_l.
//
// Attention from given features whose widths the chunk kernels do not take (d other than 32,
// 64 and 128, or more than 256 features) runs as fp32 GEMMs over 64-token chunks:
//   bwd_pack_kernel     V -> [V | 1] in fp32;
//   bwd_gemm_kernel     batched C (+)= A B over (head, chunk) with strided operands, a
//                       lower-triangular output mask and ragged last chunks;
//   bwd_scan_kernel     exclusive prefix sums of the per-chunk states, or their total;
//   fwd_out_kernel      [num | den - eps] -> out = num / den in the value type.
#include <algorithm>

#include "luna_device.hpp"
#include "luna_grad.hpp"
#include "luna_kernels.hpp"

namespace luna {

namespace {

// ---------------------------------------------------------------------------
// [V | 1] in fp32
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void bwd_pack_kernel(const T* __restrict__ V, float* __restrict__ Vx, int64_t rows,
                                                       int d) {
  const int64_t total = rows * (d + 1);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / (d + 1);
    const int c = (int)(i - r * (d + 1));
    Vx[i] = c < d ? (float)V[r * d + c] : 1.0f;
  }
}

// ---------------------------------------------------------------------------
// batched strided GEMM on the fp32 matrix cores: 64 x 64 output tiles, four waves
// of 32 x 32 (2 x 2 blocks of 16 x 16), 32-deep k slices through LDS, the next slice
// read into registers during the current slice's products.  A tile is kept
// row-major (i, k) and B transposed (j, k), so that a lane's fragment -- row (or
// column) lane % 16, k = 8 (lane / 16) + e for e < 8 -- is two 16-byte reads.  Tile
// loads let consecutive threads walk the operand's unit-stride index.
// ---------------------------------------------------------------------------
constexpr int kGT = 64, kGK = 32, kGP = kGK + 4;  // tile, k slice, LDS row (floats)

__global__ __launch_bounds__(256) void bwd_gemm_kernel(BwdGemm g) {
  __shared__ __attribute__((aligned(16))) float As[kGT][kGP];
  __shared__ __attribute__((aligned(16))) float Bt[kGT][kGP];
  const int bz = blockIdx.z;
  const int h = bz / g.chunks, c = bz - h * g.chunks;
  const int rows_left = g.seq - c * g.chunk;  // tokens of this chunk (ragged last chunk)
  const int Mv = g.m_chunk ? min(g.M, rows_left) : g.M;
  const int Nv = g.n_chunk ? min(g.N, rows_left) : g.N;
  const int Kv = g.k_chunk ? min(g.K, rows_left) : g.K;
  const float* A = g.A + h * g.sAh + c * g.sAc;
  const float* B = g.B + h * g.sBh + c * g.sBc;
  float* C = g.C + h * g.sCh + c * g.sCc;
  const int i0 = blockIdx.y * kGT, j0 = blockIdx.x * kGT;
  if (i0 >= Mv || j0 >= Nv) return;  // (uniform) tile outside this chunk's rows
  const int tid = threadIdx.x, lane = tid % kWave, wave = wave_id();
  const int grp = lane / 16, r = lane % 16;
  const int wi = 32 * (wave / 2), wj = 32 * (wave % 2);  // this wave's 32 x 32 sub-tile
  const bool a_krow = g.sAk == 1, b_jrow = g.sBj == 1;   // unit stride along k (A) or j (B)
  f32x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = zero4();
  // The next k slice is read into registers while the matrix cores work on the current
  // one from LDS, so that global-load latency overlaps the products.
  constexpr int PER = (kGK * kGT) / 256;  // elements of each operand per thread and slice
  float ra[PER], rb[PER];
  auto load_slice = [&](int k0) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int idx = tid + 256 * e;
      int ii, kk;
      if (a_krow) { kk = idx % kGK; ii = idx / kGK; }
      else { ii = idx % kGT; kk = idx / kGT; }
      const int ia = i0 + ii, ka = k0 + kk;
      ra[e] = (ka < Kv && ia < Mv) ? A[ia * g.sAi + ka * g.sAk] : 0.0f;
      int jj, kb;
      if (b_jrow) { jj = idx % kGT; kb = idx / kGT; }
      else { kb = idx % kGK; jj = idx / kGK; }
      const int jb = j0 + jj, kbb = k0 + kb;
      rb[e] = (kbb < Kv && jb < Nv) ? B[kbb * g.sBk + jb * g.sBj] : 0.0f;
    }
  };
  auto store_slice = [&]() {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int idx = tid + 256 * e;
      int ii, kk;
      if (a_krow) { kk = idx % kGK; ii = idx / kGK; }
      else { ii = idx % kGT; kk = idx / kGT; }
      As[ii][kk] = ra[e];
      int jj, kb;
      if (b_jrow) { jj = idx % kGT; kb = idx / kGT; }
      else { kb = idx % kGK; jj = idx / kGK; }
      Bt[jj][kb] = rb[e];
    }
  };
  load_slice(0);
  for (int k0 = 0; k0 < Kv; k0 += kGK) {
    store_slice();
    __syncthreads();
    if (k0 + kGK < Kv) load_slice(k0 + kGK);
    Frag<float> af[2], bf[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const float4* pa = reinterpret_cast<const float4*>(&As[wi + 16 * x + r][8 * grp]);
      const float4* pb = reinterpret_cast<const float4*>(&Bt[wj + 16 * x + r][8 * grp]);
      const float4 a0 = pa[0], a1 = pa[1], b0 = pb[0], b1 = pb[1];
      af[x].v[0] = a0.x; af[x].v[1] = a0.y; af[x].v[2] = a0.z; af[x].v[3] = a0.w;
      af[x].v[4] = a1.x; af[x].v[5] = a1.y; af[x].v[6] = a1.z; af[x].v[7] = a1.w;
      bf[x].v[0] = b0.x; bf[x].v[1] = b0.y; bf[x].v[2] = b0.z; bf[x].v[3] = b0.w;
      bf[x].v[4] = b1.x; bf[x].v[5] = b1.y; bf[x].v[6] = b1.z; bf[x].v[7] = b1.w;
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) mma(acc[x][y], af[x], bf[y]);
    __syncthreads();
  }
  // acc[x][y] holds rows 4 grp + q (q < 4), column r of block (x, y)
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + wi + 16 * x + 4 * grp + q, j = j0 + wj + 16 * y + r;
        if (i >= Mv || j >= Nv) continue;
        float v = (g.lower && j > i) ? 0.0f : acc[x][y][q];
        float* pc = C + i * g.sCi + j * g.sCj;
        if (g.accumulate) v += *pc;
        *pc = v;
      }
}

// ---------------------------------------------------------------------------
// exclusive prefix sums over chunks in place, or (total) their total in every chunk
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void bwd_scan_kernel(float* X, int heads, int chunks, int64_t elems, int total) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int h = blockIdx.y;
  if (e >= elems || h >= heads) return;
  float* base = X + (int64_t)h * chunks * elems + e;
  float run = 0.0f;
  for (int c = 0; c < chunks; ++c) {
    const float v = base[(int64_t)c * elems];
    if (!total) base[(int64_t)c * elems] = run;
    run += v;
  }
  if (total)
    for (int c = 0; c < chunks; ++c) base[(int64_t)c * elems] = run;
}

// ---------------------------------------------------------------------------
// forward readout of the generic path: out = num / (den - eps + eps), one wave per row
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void fwd_out_kernel(const float* __restrict__ Y, T* __restrict__ out, int64_t rows,
                                                      int d, float eps) {
  const int lane = threadIdx.x % kWave;
  const int64_t r = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave;
  if (r >= rows) return;
  const float* y = Y + r * (d + 1);
  const float inv = 1.0f / (y[d] + eps);
  for (int c = lane; c < d; c += kWave) out[r * d + c] = (T)(y[c] * inv);
}

// ---------------------------------------------------------------------------
// column sums in fp64: workgroups of 64 columns x 16 row lanes.  A thread takes every
// 16th row of its column (eight loads in flight), the 16 lanes of a column meet in LDS
// in a fixed order.  These sums are bound by the latency of their loads: one thread
// walking all rows of a column made the two sums of a backward call on 32 x 12 heads of
// 512 tokens (384 rows of 520 columns, 512 rows of 8208) take 101 + 186 us; with 16
// lanes the call is 279 us shorter.
// ---------------------------------------------------------------------------
constexpr int kSumCols = 64, kSumLanes = 16;

// sum over i < rows of at(i) for this thread's column; the result is valid in lane 0
template <typename F>
__device__ __forceinline__ double column_sum(int rows, F at) {
  __shared__ double part[kSumLanes][kSumCols];
  const int col = threadIdx.x % kSumCols, lane = threadIdx.x / kSumCols;
  double s = 0.0;
  int i = lane;
  for (; i + 7 * kSumLanes < rows; i += 8 * kSumLanes) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = at(i + k * kSumLanes);
#pragma unroll
    for (int k = 0; k < 8; ++k) s += (double)v[k];
  }
  for (; i < rows; i += kSumLanes) s += (double)at(i);
  part[lane][col] = s;
  __syncthreads();
  double t = 0.0;
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < kSumLanes; ++k) t += part[k][col];
  return t;
}

// ---------------------------------------------------------------------------
// [dW | db] per parameter set from the workgroups' sums [set][groups][M][d + 1]
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSumCols * kSumLanes) void bwd_dw_kernel(const float* __restrict__ partial,
                                                                      float* __restrict__ dW, float* __restrict__ db,
                                                                      int groups, int M, int d) {
  const int E = d + 1, cols = M * E, set = blockIdx.y;
  const int rest = blockIdx.x * kSumCols + threadIdx.x % kSumCols;  // (i, c)
  const float* p = partial + (size_t)set * groups * cols + min(rest, cols - 1);
  const double s = column_sum(groups, [&](int r) { return p[(size_t)r * cols]; });
  if (threadIdx.x >= kSumCols || rest >= cols) return;
  const int i = rest / E, c = rest - i * E;
  if (c < d) dW[((size_t)set * M + i) * d + c] = (float)s;
  else db[(size_t)set * M + i] = (float)s;
}

// ---------------------------------------------------------------------------
// partials summed over workgroups (fp64), per parameter set
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSumCols * kSumLanes) void bwd_reduce_kernel(const float* __restrict__ partial,
                                                                          double* __restrict__ sum, int groups,
                                                                          int part_floats, int used) {
  const int set = blockIdx.y;
  const int e = blockIdx.x * kSumCols + threadIdx.x % kSumCols;
  const float* p = partial + (size_t)set * groups * part_floats + min(e, used - 1);
  const double s = column_sum(groups, [&](int g) { return p[(size_t)g * part_floats]; });
  if (threadIdx.x < kSumCols && e < used) sum[(size_t)set * part_floats + e] = s;
}

// ---------------------------------------------------------------------------
// parameter gradients from the reduced sums
// ---------------------------------------------------------------------------

// exclusive prefix sums over segments of the moments of one channel: one workgroup
// per (channel, parameter set), a thread per segment, fp64
__global__ __launch_bounds__(1024) void bwd_prefix_kernel(const double* __restrict__ sum, double* __restrict__ pre,
                                                          const uint8_t* tables, int M, int d, int L, int part_floats,
                                                          int nseg_cap) {
  __shared__ double wtot[2][16];
  const int l = blockIdx.x, set = blockIdx.y, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const PwlHeader hd = *reinterpret_cast<const PwlHeader*>(tables + (size_t)set * kTableBytes + kTabHeader);
  const int nseg = min(max(hd.nbp, 0) + 1, nseg_cap);
  const double* mom = sum + (size_t)set * part_floats;  // [nseg][L][2]
  double* out = pre + ((size_t)set * L + l) * (nseg_cap + 1) * 2;
  double run0 = 0.0, run1 = 0.0;  // the sums of the previous 1024-segment blocks
  for (int j0 = 0; j0 <= nseg; j0 += 1024) {
    const int j = j0 + tid;
    const double v0 = j < nseg ? mom[((size_t)j * L + l) * 2] : 0.0;
    const double v1 = j < nseg ? mom[((size_t)j * L + l) * 2 + 1] : 0.0;
    double i0 = v0, i1 = v1;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const double u0 = __shfl_up(i0, o, kWave), u1 = __shfl_up(i1, o, kWave);
      if (lane >= o) {
        i0 += u0;
        i1 += u1;
      }
    }
    if (lane == kWave - 1) {
      wtot[0][wave] = i0;
      wtot[1][wave] = i1;
    }
    __syncthreads();
    double b0 = run0, b1 = run1;
    for (int w = 0; w < wave; ++w) {
      b0 += wtot[0][w];
      b1 += wtot[1][w];
    }
    if (j <= nseg) {
      out[2 * j] = b0 + i0 - v0;
      out[2 * j + 1] = b1 + i1 - v1;
    }
    double t0 = 0.0, t1 = 0.0;
    for (int w = 0; w < 16; ++w) {
      t0 += wtot[0][w];
      t1 += wtot[1][w];
    }
    run0 += t0;
    run1 += t1;
    __syncthreads();
  }
}

__device__ __forceinline__ uint32_t ordered_key(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b >> 31) ? ~b : (b | 0x80000000u);
}

__global__ __launch_bounds__(256) void bwd_mlp_kernel(BwdMlp a) {
  __shared__ float keys[kKeyCap];
  const int set = blockIdx.x, tid = threadIdx.x;
  const uint8_t* tab = a.tables + (size_t)set * kTableBytes;
  const PwlHeader hd = *reinterpret_cast<const PwlHeader*>(tab + kTabHeader);
  const int nbp = min(max(hd.nbp, 0), a.nseg_cap - 1);
  const int nseg = nbp + 1;
  const float* gkeys = reinterpret_cast<const float*>(tab + kTabKeys);
  for (int i = tid; i < nbp; i += blockDim.x) keys[i] = gkeys[i];
  const int L = a.L, hidden = a.hidden, C1 = a.C1;
  __syncthreads();
  const float* A = a.fc1_w + (size_t)set * C1 * hidden;
  const float* Cc = a.fc1_b + (size_t)set * C1 * hidden;
  const float* F = a.fc2_w + (size_t)set * L * hidden;
  const double* preset = a.pre + (size_t)set * L * (a.nseg_cap + 1) * 2;
  // sums of the moments of channel l over the segments where a unit (a, c) is on
  auto on_sums = [&](int l, float ak, float ck, double& m0, double& m1) {
    const double* P = preset + (size_t)l * (a.nseg_cap + 1) * 2;
    const float q = (float)(-(double)ck / (double)ak);
    if (ak != 0.0f && isfinite(q)) {
      // its rank: the number of keys below the breakpoint (for equal keys any of
      // them: the segments between equal keys are empty)
      const uint32_t kb = ordered_key(q == 0.0f ? 0.0f : q);
      int lo = 0, hi = nbp;
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (ordered_key(keys[mid]) < kb) lo = mid + 1;
        else hi = mid;
      }
      if (ak > 0.0f) {  // on above the breakpoint: segments j > rank
        m0 = P[2 * nseg] - P[2 * (lo + 1)];
        m1 = P[2 * nseg + 1] - P[2 * (lo + 1) + 1];
      } else {          // on below it: segments j <= rank
        m0 = P[2 * (lo + 1)];
        m1 = P[2 * (lo + 1) + 1];
      }
    } else if (ck > 0.0f) {  // constant and on
      m0 = P[2 * nseg];
      m1 = P[2 * nseg + 1];
    } else {
      m0 = m1 = 0.0;
    }
  };
  for (int idx = tid; idx < L * hidden; idx += blockDim.x) {
    const int l = idx / hidden, k = idx - l * hidden;
    const int u = (C1 == 1 ? 0 : l) * hidden + k;
    double m0, m1;
    on_sums(l, A[u], Cc[u], m0, m1);
    a.dfc2_w[(size_t)set * L * hidden + idx] = (float)((double)A[u] * m1 + (double)Cc[u] * m0);
  }
  for (int l = tid; l < L; l += blockDim.x)
    a.dfc2_b[(size_t)set * L + l] = (float)preset[((size_t)l * (a.nseg_cap + 1) + nseg) * 2];
  for (int u = tid; u < C1 * hidden; u += blockDim.x) {
    const int k = u % hidden;
    const int l0 = C1 == 1 ? 0 : u / hidden, l1 = C1 == 1 ? L : u / hidden + 1;
    double g1 = 0.0, g0 = 0.0;
    for (int l = l0; l < l1; ++l) {
      double m0, m1;
      on_sums(l, A[u], Cc[u], m0, m1);
      const double f = (double)F[l * hidden + k];
      g1 += f * m1;
      g0 += f * m0;
    }
    a.dfc1_w[(size_t)set * C1 * hidden + u] = (float)g1;
    a.dfc1_b[(size_t)set * C1 * hidden + u] = (float)g0;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_bwd_pack(Dt dt, const void* V, float* Vx, int64_t rows, int d, hipStream_t s) {
  const int64_t total = rows * (d + 1);
  const dim3 grid((unsigned)std::min<int64_t>((total + 255) / 256, 65536)), block(256);
  if (dt == Dt::BF16) hipLaunchKernelGGL(bwd_pack_kernel<__bf16>, grid, block, 0, s, (const __bf16*)V, Vx, rows, d);
  else hipLaunchKernelGGL(bwd_pack_kernel<float>, grid, block, 0, s, (const float*)V, Vx, rows, d);
  return hipGetLastError();
}

hipError_t launch_bwd_gemm(const BwdGemm& g, hipStream_t s) {
  // at most 65535 (head, chunk) batches per launch: whole heads per slice
  const int per = std::max(1, 65535 / std::max(1, g.chunks));
  for (int h0 = 0; h0 < g.heads; h0 += per) {
    BwdGemm q = g;
    q.heads = std::min(per, g.heads - h0);
    q.A = g.A + h0 * g.sAh;
    q.B = g.B + h0 * g.sBh;
    q.C = g.C + h0 * g.sCh;
    const dim3 grid((unsigned)((g.N + kGT - 1) / kGT), (unsigned)((g.M + kGT - 1) / kGT),
                    (unsigned)(q.heads * g.chunks));
    hipLaunchKernelGGL(bwd_gemm_kernel, grid, dim3(256), 0, s, q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_bwd_scan(float* X, int heads, int chunks, int64_t elems, bool total, hipStream_t s) {
  for (int h0 = 0; h0 < heads; h0 += 65535) {  // at most 65535 heads per launch
    const int hn = std::min(65535, heads - h0);
    const dim3 grid((unsigned)((elems + 255) / 256), (unsigned)hn);
    hipLaunchKernelGGL(bwd_scan_kernel, grid, dim3(256), 0, s, X + (int64_t)h0 * chunks * elems, hn, chunks, elems,
                       total);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool bwd_supported(int d, int L, int M) {
  const bool lok = L == 1 || L == 2 || L == 4 || L == 8 || L == 16;
  return lok && M >= 1 && M <= 256 && M * L <= 256 && d >= 1 && d <= 128;
}

size_t bwd_part_floats(int, int L, int) { return 2 * (size_t)nseg_cap(L, kFmSegBytes) * L; }

hipError_t launch_bwd_dw(const float* partial, float* dW, float* db, int groups, int M, int d, int sets,
                         hipStream_t s) {
  const dim3 grid((unsigned)((M * (d + 1) + kSumCols - 1) / kSumCols), (unsigned)sets);
  hipLaunchKernelGGL(bwd_dw_kernel, grid, dim3(kSumCols * kSumLanes), 0, s, partial, dW, db, groups, M, d);
  return hipGetLastError();
}

hipError_t launch_bwd_reduce(const float* partial, double* sum, int groups, int part_floats, int used, int sets,
                             hipStream_t s) {
  const dim3 grid((unsigned)((used + kSumCols - 1) / kSumCols), (unsigned)sets);
  hipLaunchKernelGGL(bwd_reduce_kernel, grid, dim3(kSumCols * kSumLanes), 0, s, partial, sum, groups, part_floats, used);
  return hipGetLastError();
}

hipError_t launch_bwd_prefix(const double* sum, double* pre, const uint8_t* tables, int M, int d, int L,
                             int part_floats, int nseg_cap_, int sets, hipStream_t s) {
  hipLaunchKernelGGL(bwd_prefix_kernel, dim3((unsigned)L, (unsigned)sets), dim3(1024), 0, s, sum, pre, tables, M, d, L,
                     part_floats, nseg_cap_);
  return hipGetLastError();
}

hipError_t launch_bwd_mlp(const BwdMlp& a, int sets, hipStream_t s) {
  hipLaunchKernelGGL(bwd_mlp_kernel, dim3((unsigned)sets), dim3(256), 0, s, a);
  return hipGetLastError();
}

int bwd_nseg_cap(int L) { return nseg_cap(L, kFmSegBytes); }

hipError_t launch_fwd_out(Dt dt, const float* Y, void* out, int64_t rows, int d, float eps, hipStream_t s) {
  const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  if (dt == Dt::BF16) hipLaunchKernelGGL(fwd_out_kernel<__bf16>, grid, block, 0, s, Y, (__bf16*)out, rows, d, eps);
  else hipLaunchKernelGGL(fwd_out_kernel<float>, grid, block, 0, s, Y, (float*)out, rows, d, eps);
  return hipGetLastError();
}

}  // namespace luna
