// luna_chunk_query.hip -- the query pass of the chunked attention kernel and the scan of the
// pieces' states.
#include "luna_chunk_kernel.hpp"

namespace luna {

namespace {

// A thread takes one element of a head's states through the pieces, eight loads in flight.
template <bool SUFFIX>
__global__ __launch_bounds__(256) void chunk_scan_kernel(float* state, int64_t heads, int pieces, int64_t elems) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= heads * elems) return;
  const int64_t h = i / elems;
  float* p = state + h * pieces * elems + (i - h * elems);
  auto at = [&](int c) -> float& { return p[(int64_t)(SUFFIX ? pieces - 1 - c : c) * elems]; };
  float run = 0.0f;
  int c = 0;
  for (; c + 8 <= pieces; c += 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = at(c + k);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      at(c + k) = run;
      run += v[k];
    }
  }
  for (; c < pieces; ++c) {
    const float v = at(c);
    at(c) = run;
    run += v;
  }
}

}  // namespace

bool chunk_supported(int d, int D) { return (d == 32 || d == 64 || d == 128) && D >= 1 && D <= 256; }

hipError_t launch_chunk_query(Dt dt, int d, const ChunkArgs& a, hipStream_t s) {
  return chunk_launch_p<kPassQuery>(dt, d, a, s);
}

hipError_t launch_chunk_scan(float* state, int64_t heads, int pieces, int64_t elems, bool suffix, hipStream_t s) {
  return by_heads(heads, elems + 256, [&](int64_t h0, int64_t hn) {
    const dim3 grid((unsigned)((hn * elems + 255) / 256)), block(256);
    float* at = state + h0 * pieces * elems;
    if (suffix) hipLaunchKernelGGL(chunk_scan_kernel<true>, grid, block, 0, s, at, hn, pieces, elems);
    else hipLaunchKernelGGL(chunk_scan_kernel<false>, grid, block, 0, s, at, hn, pieces, elems);
    return hipGetLastError();
  });
}

}  // namespace luna
