// luna_features.hpp -- host interface of attention from features in memory
// (luna_features.hip).
#pragma once

#include "luna_kernels.hpp"

namespace luna {

// Statistics of a piece of a head's tokens: S [D][d], then z [D], fp32, `elems` floats apart.
struct FeatArgs {
  const void* phiq;   // [heads][n][D], feature type
  const void* phik;
  const void* v;      // [heads][n][d], value type
  void* out;          // [heads][n][d], value type
  float* state;       // [heads][pieces] statistics
  const float* w;     // [heads][n][2] or null: S = (w0 phi(K))^T V, z = phi(K)^T w1
  int64_t heads, n, elems;
  int D, piece, pieces;  // tokens per piece (a multiple of 32) and pieces per head
  int tokens;            // readout: tokens per workgroup (set by the launcher)
  float eps;
};

bool feat_supported(int d, int D);
// floats from one piece's statistics to the next's: whole 16-byte rows of S
constexpr int64_t feat_elems(int64_t d, int64_t D) { return (D * (d + 1) + 3) / 4 * 4; }
// features per workgroup of the state kernel: all of them in blocks of 64, or half or a quarter
// while the pieces' workgroups still find a compute unit each
constexpr int feat_state_features(int D, int64_t pieces) {
  int each = D <= 64 ? 64 : D <= 128 ? 128 : 256;
  while (each > 64 && pieces * ((D + each / 2 - 1) / (each / 2)) <= 256) each /= 2;
  return each;
}
// per piece: S = phi(K)^T V, z = phi(K)^T 1
hipError_t launch_feat_state(Dt fdt, Dt vdt, int d, const FeatArgs& a, hipStream_t s);
// the pieces of every head summed into its first (in order)
hipError_t launch_feat_total(const FeatArgs& a, hipStream_t s);
// out = phi(Q) S / (phi(Q) z + eps) with each head's first piece as its statistics
hipError_t launch_feat_readout(Dt fdt, Dt vdt, int d, const FeatArgs& a, hipStream_t s);
// each head's first piece into (or added to) S [heads][D][d] and z [heads][D]
hipError_t launch_feat_export(int d, const FeatArgs& a, float* S, float* z, int accumulate, hipStream_t s);

}  // namespace luna
