// luna_chunk.hpp -- host interface of the fp32 chunked attention kernels
// (luna_chunk_query.hip, luna_chunk_key.hip): the causal forward of shapes without a fused
// kernel and the attention part of the backward pass.
#pragma once

#include "luna_kernels.hpp"

namespace luna {

constexpr int kChunkTile = 64;  // tokens per workgroup

// "rows" are the tokens a workgroup owns, "columns" the tokens it meets in its piece:
// queries and keys in the query pass, keys and queries in the key pass.
struct ChunkArgs {
  const float* x;      // row features [heads][n][D]
  const void* u;       // row values [heads][n][d]: dO (query pass), V (key pass); null: forward
  const float* y;      // column features
  const void* v;       // column values: V (query pass), dO (key pass)
  const float* state;  // [heads][pieces][elems]: S [D][d] then z [D] outside the piece (causal), or the total
  float* w;            // [heads][n][2]: 1 / den and dden, written by the query pass, read by the key pass
  void* out;           // forward: out; key pass: dV ([heads][n][d], value type)
  float* dx;           // row feature gradients [heads][n][D]
  int64_t heads, n, elems;
  int D, piece, pieces, causal;  // tokens per piece (a multiple of the tile), pieces per head
  int first, step;               // tiles first, first + step, ... of every head (set by the launcher)
  float eps;
};

// Tokens per piece of the causal form.  Every piece's state is written once, scanned in place
// and read twice or more, while a tile also meets the other tiles of its piece.  Backward of
// 2 x 16 heads of 2048 tokens, d = 128, D = 256: states and scans take 210 us at one tile a
// piece and 139 us at two, the query and key passes 350 and 401 us.  Calls with one, two and
// four tiles a piece, 32 heads of 1024 tokens: that backward 415 / 404 / 462 us, with D = 128
// 263 / 273 / 330, in fp32 497 / 497 / 584 and 327 / 339 / 410; d = 64, D = 128 193 / 204 / 246;
// the fp32 forward with D = 256 166 / 158 / 177, with 128 106 / 104 / 118.  4 heads of 333
// tokens: 186 / 206 / 252 and 57 / 64 / 83.  (Two suit the largest maps and the forward, one
// the smaller maps' backward and short calls.)
constexpr int kChunkPiece = 128;

bool chunk_supported(int d, int D);
// forward (u == null): out = num / den; else den and dphi(Q)
hipError_t launch_chunk_query(Dt dt, int d, const ChunkArgs& a, hipStream_t s);
// dphi(K) and dV
hipError_t launch_chunk_key(Dt dt, int d, const ChunkArgs& a, hipStream_t s);
// exclusive prefix (suffix: of the pieces after) sums over the pieces of every head, in place
hipError_t launch_chunk_scan(float* state, int64_t heads, int pieces, int64_t elems, bool suffix, hipStream_t s);

}  // namespace luna
