// luna_api.cpp -- host side of the C ABI declared in include/luna.h.
//
// Every entry point validates its arguments completely on the host before any HIP
// call, plans the workspace (piecewise-linear tables first, then per-operation
// buffers, each 256-byte aligned) and enqueues its kernels on the caller's stream.
#include "luna.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <string>

#include "luna_chunk.hpp"
#include "luna_features.hpp"
#include "luna_grad.hpp"
#include "luna_kernels.hpp"

namespace {

thread_local std::string g_last_error;

luna_status fail(luna_status s, const std::string& why) {
  g_last_error = why;
  return s;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct Problem {
  int op;
  luna_dtype dt;
  int64_t B, H, n, d;
  const luna_phi_params* p;
  int32_t chunk;
};

int param_sets(const Problem& pb) { return pb.p->per_head ? (int)pb.H : 1; }

// Checks shared by every operation; `why` receives the reason on failure.
luna_status check_common(const Problem& pb) {
  const luna_phi_params* p = pb.p;
  if (p == nullptr) return fail(LUNA_ERR_INVALID_ARG, "params is NULL");
  if (pb.dt != LUNA_F32 && pb.dt != LUNA_BF16) return fail(LUNA_ERR_INVALID_ARG, "dtype must be LUNA_F32 or LUNA_BF16");
  if (pb.B < 1 || pb.H < 1 || pb.n < 1) return fail(LUNA_ERR_INVALID_ARG, "B, H and n must be >= 1");
  if (pb.n > (int64_t)1 << 30) return fail(LUNA_ERR_UNSUPPORTED, "n must be <= 2^30");
  if (pb.B * pb.H > (int64_t)1 << 24) return fail(LUNA_ERR_UNSUPPORTED, "B*H must be <= 2^24");
  if (pb.d != 32 && pb.d != 64 && pb.d != 128) return fail(LUNA_ERR_UNSUPPORTED, "d must be 32, 64 or 128");
  if (p->M < 1 || p->M > 256) return fail(LUNA_ERR_INVALID_ARG, "M must be in [1, 256]");
  if (p->L < 1 || p->L > 16) return fail(LUNA_ERR_INVALID_ARG, "L must be in [1, 16]");
  if (p->hidden < 1 || p->hidden > 64) return fail(LUNA_ERR_INVALID_ARG, "hidden must be in [1, 64]");
  if (p->M * p->L > 256) return fail(LUNA_ERR_INVALID_ARG, "M*L must be <= 256");
  if (p->shared_channels != 0 && p->shared_channels != 1) return fail(LUNA_ERR_INVALID_ARG, "shared_channels must be 0 or 1");
  if (p->nonneg != 0 && p->nonneg != 1) return fail(LUNA_ERR_INVALID_ARG, "nonneg must be 0 or 1");
  if (p->per_head != 0 && p->per_head != 1) return fail(LUNA_ERR_INVALID_ARG, "per_head must be 0 or 1");
  if (!p->W || !p->b || !p->fc1_w || !p->fc1_b || !p->fc2_w || !p->fc2_b)
    return fail(LUNA_ERR_INVALID_ARG, "a parameter array is NULL");
  const int C1 = p->shared_channels ? 1 : p->L;
  const int units = C1 * p->hidden;
  if (units > luna::kMaxUnits) return fail(LUNA_ERR_UNSUPPORTED, "L*hidden must be <= 1023 (breakpoint table)");
  // the feature-map kernel (also the first stage of a streaming step) has the larger LDS table
  const bool fm_table = pb.op == LUNA_OP_FEATUREMAP || pb.op == LUNA_OP_CAUSAL_STEP || pb.op == LUNA_OP_ATTN_BWD ||
                        pb.op == LUNA_OP_ATTN_CAUSAL_BWD || pb.op >= 100;
  const int seg_cap = luna::nseg_cap(p->L, fm_table ? luna::kFmSegBytes : luna::kAttnSegBytes);
  if (units + 2 > seg_cap) return fail(LUNA_ERR_UNSUPPORTED, "too many breakpoints for the LDS segment table");
  if ((units + 1) * p->L > luna::kSegCap || (size_t)(units + 1) * luna::seg16_row_bytes(p->L) > luna::kSeg16Bytes)
    return fail(LUNA_ERR_UNSUPPORTED, "too many segments for the table");
  return LUNA_OK;
}

struct Layout {
  size_t tables = 0, partial = 0, frags = 0, total = 0;
  size_t phiq = 0, phik = 0;  // streaming step: features of the new queries and keys (fp32)
  size_t zcopy = 0;           // streaming step: z as it was before the call
  // backward pass: per-piece states and their gradients, per query [1 / den, dden],
  // feature gradients, per-workgroup parameter partials, their fp64 sums and moment
  // prefixes; fp32 forward of given features by GEMMs: [V | 1], [num | den - eps], states, P
  size_t sx = 0, dsx = 0, wq = 0, dphiq = 0, dphik = 0, vx = 0, y = 0, pm = 0;
  size_t duq = 0, duk = 0, dwp = 0;  // feature-map backward
  size_t bpart = 0, sum = 0, pre = 0;
  size_t dstats = 0;  // distillation: per query row the softmax max and sum and the kernel row sum
  int chunk = 0, nch = 1, groups = 0, dw_groups = 0, part_floats = 0;
  int splits = 1, tokens_per_split = 0, tile_tokens = 256, tiles = 1, fused = 0;
  int parts = 1, split = 0;  // causal: workgroups per head, first token of part 1 (of the last of equal parts)
  int part_chunks = 0;       // chunks of equal parts
  size_t state_floats = 0;   // floats per state piece
  size_t state = 0;          // causal with 2 parts: state pieces of the first `split` tokens
  int pieces = 0, piece_chunks = 0;
  int staged = 0, sa = 0, sb = 0;  // staged causal scan: chunks of the first scanned part and of the state-only part
  bool few = false;  // the plan of a small workspace: statistics in as few pieces as it can
  int feat = 0;     // non-causal attention from given features in their own type
  int generic = 0;  // forward in fp32 (shapes without a fused kernel),
  int chunked = 0;  // by the chunk kernels; else by GEMMs and scans
  int given = 0;    // causal: features mapped beforehand (bf16, in phiq / phik), then the scan kernel
};

// Tokens per piece of the statistics of a whole sequence: 512, or fewer (64 at least) while
// there are not enough pieces for the compute units and the shorter chain pays.  A piece is a
// serial chain of 32-token steps: with fp32 features and values 4.9 us a step at 256 features in
// one workgroup and d = 128, 1.5 at 128 and 64, 0.6 at 64 and 32; in bf16 1.4, 0.55 and 0.3; the
// two mixed in between.  Cut, it takes a launch that adds up the pieces (3 us) and every piece's
// state written and read (5.8 TB/s).  256 features, d = 128, one piece of the whole against
// pieces of 64, us a call: fp32, 1 head of 512 tokens 44 / 28, bf16 23.4 / 21.6; 64 bf16 heads of
// 100 tokens 17 / 33, 128 fp32 heads of 100 tokens 36 / 51.
int state_piece(luna::Dt fdt, luna::Dt vdt, int64_t heads, int64_t n, int d, int D, bool few) {
  const double elems = (double)luna::feat_elems(d, D);
  const bool mixed = fdt != vdt, bf16 = fdt == luna::Dt::BF16;
  const double each_step = mixed ? 0.25 : bf16 ? 0.22 : 0.3, each_elem = mixed ? 7e-5 : bf16 ? 3.6e-5 : 1.4e-4;
  auto cost = [&](int64_t piece) {  // us
    const int64_t pieces = (n + piece - 1) / piece, steps = (std::min(n, piece) + 31) / 32;
    const double part = std::min(1.0, (double)luna::feat_state_features(D, heads * pieces) / D);
    return steps * (each_step + each_elem * elems * part) + (pieces > 1 ? 3.0 + 1.4e-6 * elems * heads * pieces : 0.0);
  };
  int best = 512;
  for (int piece = 256; !few && piece >= 64 && heads * ((n + 2 * piece - 1) / (2 * piece)) < 256; piece /= 2)
    if (cost(piece) < cost(best)) best = piece;
  return best;
}

// Buffers of the forward pass in fp32 (the forward of shapes without a fused kernel, and
// the start of the backward pass): features of the keys (and queries) and the statistics of
// pieces of the tokens.  Causal pieces are a few tiles long (luna_chunk.hpp), the
// non-causal form cuts its sums over tokens into pieces for parallelism only.
// Widths that only given features have take fp32 GEMMs over 64-token chunks: [V | 1],
// [num | den - eps] and the per-chunk states, plus P for the causal form.
// (features: the buffers for fp32 features, or none when the caller's are used)
luna_status plan_f32_buffers(luna::Dt vdt, int64_t heads, int64_t n, int d, int D, bool causal, bool queries,
                             bool features, Layout* lay, size_t* off) {
  lay->chunk = causal ? 64 : 512;
  int64_t nch = (n + lay->chunk - 1) / lay->chunk;
  if (nch > 65535) return fail(LUNA_ERR_UNSUPPORTED, causal ? "n must be <= 65535 * 64" : "n must be <= 65535 * 512");
  lay->chunked = luna::chunk_supported(d, D);
  if (lay->chunked) {
    lay->chunk = causal ? luna::kChunkPiece
                        : state_piece(luna::Dt::F32, vdt, heads, n, d, D, lay->few);
    nch = (n + lay->chunk - 1) / lay->chunk;
  }
  lay->nch = (int)nch;
  const size_t rows = (size_t)heads * (size_t)n, states = (size_t)heads * lay->nch;
  auto take = [&](size_t& at, size_t bytes) {
    at = *off;
    *off = align256(*off + bytes);
  };
  if (queries && features) take(lay->phiq, rows * D * 4);
  if (features) take(lay->phik, rows * D * 4);
  if (lay->chunked) {
    take(lay->sx, states * (size_t)luna::feat_elems(d, D) * 4);
    return LUNA_OK;
  }
  take(lay->vx, rows * (d + 1) * 4);
  if (queries) take(lay->y, rows * (d + 1) * 4);
  take(lay->sx, states * D * (d + 1) * 4);
  if (causal && queries) take(lay->pm, states * 64 * 64 * 4);
  return LUNA_OK;
}
luna_status plan_f32_forward(const Problem& pb, bool causal, bool queries, Layout* lay, size_t* off) {
  return plan_f32_buffers(pb.dt == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, pb.B * pb.H, pb.n, (int)pb.d,
                          pb.p->M * pb.p->L, causal, queries, true, lay, off);
}

// The causal kernel's split.  Too few heads to fill the device: up to 85 heads in equal parts
// (short sequences in one), with 97 to 128 heads the staged form below (two scan launches);
// otherwise cut every head in two at a chunk boundary x near n/2, where a state launch first
// sums the state of [0, x) in pieces (one workgroup per head and piece, enough pieces to fill
// the device) and part 1 of the scan launch starts from the sum of the pieces.
void plan_causal_parts(luna::Dt dt, int64_t heads, int64_t n, size_t state_floats, Layout* lay, size_t* off,
                       bool staged_ok) {
  const int64_t nch = (n + 63) / 64;
  lay->state_floats = state_floats;
  // the cut in two: chunks before it, chunks of a piece, pieces
  const int64_t cx = heads < 256 && n >= 256 ? n / 64 / 2 : 0;
  int64_t pc = 0, pieces = 0;
  if (cx > 0) {
    pieces = std::min((256 + heads - 1) / heads, cx);
    pc = (cx + pieces - 1) / pieces;
    pieces = (cx + pc - 1) / pc;  // every piece non-empty
  }
  if (heads <= 85) {
    // Equal parts: a state launch over all but the last, their running sums, one scan
    // launch, for a chain of one part in place of a cut's n / 2 tokens (16 heads of 32 chunks,
    // d = 128, 32 projections in bf16: 61 us a call, 222 cut in two).  The two further
    // launches and the states cost what some chunks of a chain do, the more the more heads.
    // One part against equal parts, the same map: 1 head 39 / 38 us at 6 chunks, 31 / 38 at 4;
    // 16 heads 39 / 47 at 6, 47 / 51 at 8, 56 / 52 at 10; 64 heads 56 / 63 at 10, 80 / 69 at
    // 16.  In fp32 a chunk takes twice the time: d = 64, 16 projections, 1 head 39 / 37 at 3
    // chunks, 64 heads 39 / 42 at 3 and 47 / 44 at 4.
    if (nch < (dt == luna::Dt::BF16 ? 6 + heads / 12 : 3 + heads / 40)) return;
    // With a small workspace no more states than the cut in two would hold.
    int64_t parts = std::min(256 / heads, nch);
    if (lay->few) parts = std::min(parts, pieces + 1);
    if (parts == 1) return;
    pc = (nch + parts - 1) / parts;
    lay->part_chunks = lay->piece_chunks = (int)pc;
    lay->parts = (int)((nch + pc - 1) / pc);
    lay->pieces = lay->parts - 1;
    lay->split = (int)(64 * pc * lay->pieces);
    lay->state = *off;
    *off = align256(*off + (size_t)heads * lay->pieces * state_floats * sizeof(float));
    return;
  }
  if (staged_ok && heads > 96 && heads <= 128 && nch >= 5) {
    // Two workgroups per head fill the device, so both launches are scan launches
    // (staged): the first scans chunks [0, A) of every head and, beside it, sums the
    // state of [A, A + B); the second scans [A, A + B) and [A + B, nch) from those
    // states.  A state-only chunk costs about half a scanned one, so A = nch / 5 and
    // B = C = 2 nch / 5 balance both launches (about 153 scanned-chunk times for 256
    // chunks, against 161 for a state launch over [0, nch / 2) followed by two
    // scanned halves).
    const int64_t A = (nch + 2) / 5;
    const int64_t B = (nch - A) / 2;
    lay->parts = 2;
    lay->staged = 1;
    lay->sa = (int)A;
    lay->sb = (int)B;
    lay->split = (int)(64 * A);
    lay->pieces = 2;
    lay->piece_chunks = 0;
    lay->state = *off;
    *off = align256(*off + (size_t)heads * 2 * state_floats * sizeof(float));
    return;
  }
  if (cx > 0) {
    lay->parts = 2;
    lay->split = (int)(cx * 64);
    lay->piece_chunks = (int)pc;
    lay->pieces = (int)pieces;
    lay->state = *off;
    *off = align256(*off + (size_t)heads * lay->pieces * state_floats * sizeof(float));
  }
}

// Token ranges of the non-causal state pass: enough state workgroups to fill the
// device, at least 256 tokens each, a multiple of 128 tokens per range.  Where that leaves
// at most a quarter of the compute units at work, 128 tokens: a workgroup's time is then its
// own serial chain.
void plan_splits(const Problem& pb, int64_t heads, Layout* lay) {
  const int64_t want = (512 + heads - 1) / heads;
  const int64_t least = !lay->few && heads * ((pb.n + 255) / 256) <= 64 ? 128 : 256;
  const int64_t maxs = (pb.n + least - 1) / least;
  int64_t splits = want < maxs ? want : maxs;
  if (splits < 1) splits = 1;
  int64_t tps = (pb.n + splits - 1) / splits;
  tps = (tps + 127) / 128 * 128;
  splits = (pb.n + tps - 1) / tps;
  lay->splits = (int)splits;
  lay->tokens_per_split = (int)tps;
}

// Private operation codes of the distillation loss (without and with the feature-map
// parameter gradients).
constexpr int kOpDistill = 100, kOpDistillGrads = 101;

// Buffers of the feature-map backward (enqueue_phi_backward): the projections'
// gradients, per-workgroup [dW | db] and moments, the moments' fp64 sums and prefixes.
void plan_phi_backward(const Problem& pb, Layout* lay, size_t* off) {
  const int d = (int)pb.d, L = pb.p->L, M = pb.p->M, P = param_sets(pb);
  const int64_t heads = pb.B * pb.H, rows_per_set = pb.n * (heads / P);
  const size_t rows = (size_t)heads * (size_t)pb.n;
  auto take = [&](size_t& at, size_t bytes) {
    at = *off;
    *off = align256(*off + bytes);
  };
  take(lay->duq, rows * M * 4);
  take(lay->duk, rows * M * 4);
  lay->groups = luna::map_bwd_groups(rows_per_set, P);
  lay->dw_groups = luna::map_dw_groups(rows_per_set, P);
  lay->part_floats = (int)luna::bwd_part_floats(d, L, M);
  take(lay->dwp, (size_t)P * lay->dw_groups * M * (d + 1) * 4);
  take(lay->bpart, (size_t)P * lay->groups * lay->part_floats * 4);
  take(lay->sum, (size_t)P * lay->part_floats * 8);
  take(lay->pre, (size_t)P * L * (luna::bwd_nseg_cap(L) + 1) * 2 * 8);
}

// The plan that `f` makes: with a workspace of `room` bytes that does not hold it, the one with
// as few pieces as the call can do with (the same sums over tokens in fewer parts, slower).
template <typename F>
luna_status plan_within(size_t room, Layout* lay, F f) {
  const luna_status st = f(lay);
  if (st != LUNA_OK || lay->total <= room) return st;
  *lay = Layout();
  lay->few = true;
  return f(lay);
}

luna_status plan_pieces(const Problem& pb, Layout* lay) {
  luna_status st = check_common(pb);
  if (st != LUNA_OK) return st;
  const luna::Dt dt = pb.dt == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  const int d = (int)pb.d, L = pb.p->L, M = pb.p->M;
  const int64_t heads = pb.B * pb.H;
  size_t off = 0;
  lay->tables = off;
  off = align256(off + (size_t)param_sets(pb) * luna::kTableBytes);
  if (pb.op == LUNA_OP_FEATUREMAP) {
    if (!luna::featuremap_supported(dt, d, L, M))
      return fail(LUNA_ERR_UNSUPPORTED, "no feature-map kernel for this (d, L, M)");
  } else if (pb.op == LUNA_OP_ATTN) {
    luna::NoncausalPlan np;
    if (!luna::noncausal_supported(dt, d, L, M, &np)) {
      if (!luna::featuremap_supported(dt, d, L, M))
        return fail(LUNA_ERR_UNSUPPORTED, "no non-causal attention kernels for this (dtype, d, L, M)");
      lay->generic = 1;
      if ((st = plan_f32_forward(pb, false, true, lay, &off)) != LUNA_OK) return st;
      lay->total = off;
      return LUNA_OK;
    }
    if (heads >= luna::kFusedMinHeads && luna::fused_acc_regs(d, L, M) <= luna::kFusedMaxAccRegs) {
      lay->fused = 1;
      lay->total = off;
      return LUNA_OK;
    }
    plan_splits(pb, heads, lay);
    // 256 tokens a readout workgroup, or 64 (one block of 16 per wave) while one round of
    // workgroups then still does (1 head of 256 fp32 tokens, d = 32: 7 us instead of 14)
    lay->tile_tokens = heads * ((pb.n + 63) / 64) <= 256 ? 64 : 256;
    lay->tiles = (int)((pb.n + lay->tile_tokens - 1) / lay->tile_tokens);
    lay->partial = off;
    off = align256(off + (size_t)heads * lay->splits * np.DP * (d + 1) * sizeof(float));
    lay->frags = off;
    off = align256(off + (size_t)heads * np.frag_elems * (pb.dt == LUNA_BF16 ? 2 : 4));
  } else if (pb.op == LUNA_OP_ATTN_CAUSAL) {
    if (pb.chunk != 64) return fail(LUNA_ERR_UNSUPPORTED, "chunk must be 64");
    size_t state_floats = 0;
    if (luna::causal_supported(dt, d, L, M)) {
      state_floats = luna::causal_state_floats(dt, d, L, M);
    } else if (!luna::featuremap_supported(dt, d, L, M)) {
      return fail(LUNA_ERR_UNSUPPORTED, "no causal attention kernels for this (dtype, d, L, M)");
    } else if (luna::causal_given_supported(dt, d, M * L)) {
      // the features of Q and K in bf16, mapped by the feature-map kernel
      lay->given = 1;
      state_floats = luna::causal_given_state_floats(d, M * L);
      const size_t feat_bytes = (size_t)heads * (size_t)pb.n * (size_t)(M * L) * 2;
      lay->phiq = off;
      off = align256(off + feat_bytes);
      lay->phik = off;
      off = align256(off + feat_bytes);
    } else {
      lay->generic = 1;
      if ((st = plan_f32_forward(pb, true, true, lay, &off)) != LUNA_OK) return st;
      lay->total = off;
      return LUNA_OK;
    }
    plan_causal_parts(dt, heads, pb.n, state_floats, lay, &off, !lay->given);
  } else if (pb.op == LUNA_OP_STATE) {
    luna::NoncausalPlan np;
    if (luna::noncausal_supported(dt, d, L, M, &np)) {
      // the state pass of the non-causal split path
      plan_splits(pb, heads, lay);
      lay->partial = off;
      off = align256(off + (size_t)heads * lay->splits * np.DP * (d + 1) * sizeof(float));
    } else if (luna::causal_supported(dt, d, L, M)) {
      // the causal kernel's state launch over every chunk, in pieces
      const int64_t cx = (pb.n + 63) / 64;
      int64_t pieces = (256 + heads - 1) / heads;
      if (pieces > cx) pieces = cx;
      const int64_t pc = (cx + pieces - 1) / pieces;
      lay->piece_chunks = (int)pc;
      lay->pieces = (int)((cx + pc - 1) / pc);
      lay->split = (int)(cx * 64);
      lay->state = off;
      off = align256(off + (size_t)heads * lay->pieces * luna::causal_state_floats(dt, d, L, M) * sizeof(float));
    } else if (luna::featuremap_supported(dt, d, L, M)) {
      lay->generic = 1;
      if ((st = plan_f32_forward(pb, false, false, lay, &off)) != LUNA_OK) return st;
    } else {
      return fail(LUNA_ERR_UNSUPPORTED, "no state kernels for this (dtype, d, L, M)");
    }
  } else if (pb.op == LUNA_OP_CAUSAL_STEP) {
    if (!luna::featuremap_supported(dt, d, L, M))
      return fail(LUNA_ERR_UNSUPPORTED, "no feature-map kernel for this (d, L, M)");
    const size_t feat_bytes = (size_t)heads * (size_t)pb.n * (size_t)(M * L) * sizeof(float);
    lay->phiq = off;
    off = align256(off + feat_bytes);
    lay->phik = off;
    off = align256(off + feat_bytes);
    lay->zcopy = off;
    off = align256(off + (size_t)heads * (size_t)(M * L) * sizeof(float));
  } else if (pb.op == LUNA_OP_ATTN_BWD || pb.op == LUNA_OP_ATTN_CAUSAL_BWD) {
    if (!luna::bwd_supported(d, L, M) || !luna::featuremap_supported(dt, d, L, M))
      return fail(LUNA_ERR_UNSUPPORTED, "no backward kernels for this (d, L, M)");
    const int64_t P = param_sets(pb);
    if (P > 65535) return fail(LUNA_ERR_UNSUPPORTED, "at most 65535 parameter sets in the backward pass");
    if (pb.H > 65535) return fail(LUNA_ERR_UNSUPPORTED, "at most 65535 heads in the backward pass");
    const bool causal = pb.op == LUNA_OP_ATTN_CAUSAL_BWD;
    if ((st = plan_f32_forward(pb, causal, true, lay, &off)) != LUNA_OK) return st;
    const size_t D = (size_t)M * L, rows = (size_t)heads * (size_t)pb.n, states = (size_t)heads * lay->nch;
    auto take = [&](size_t& at, size_t bytes) {
      at = off;
      off = align256(off + bytes);
    };
    take(lay->dsx, states * (size_t)luna::feat_elems(d, D) * 4);
    take(lay->wq, rows * 2 * 4);
    take(lay->dphiq, rows * D * 4);
    take(lay->dphik, rows * D * 4);
    plan_phi_backward(pb, lay, &off);
  } else if (pb.op == kOpDistill || pb.op == kOpDistillGrads) {
    const int D = M * L;
    if (!luna::distill_supported(dt, d, D) || !luna::featuremap_supported(dt, d, L, M))
      return fail(LUNA_ERR_UNSUPPORTED, "no distillation kernels for this (dtype, d, M*L)");
    const size_t rows = (size_t)heads * (size_t)pb.n;
    auto take = [&](size_t& at, size_t bytes) {
      at = off;
      off = align256(off + bytes);
    };
    take(lay->phiq, rows * D * (pb.dt == LUNA_BF16 ? 2 : 4));  // features in the call's dtype
    take(lay->phik, rows * D * (pb.dt == LUNA_BF16 ? 2 : 4));
    take(lay->dstats, rows * 4 * sizeof(float));
    if (pb.op == kOpDistillGrads) {
      if (!luna::bwd_supported(d, L, M)) return fail(LUNA_ERR_UNSUPPORTED, "no backward kernels for this (d, L, M)");
      if (param_sets(pb) > 65535 || pb.H > 65535)
        return fail(LUNA_ERR_UNSUPPORTED, "at most 65535 heads and parameter sets in the backward pass");
      take(lay->dphiq, rows * D * 4);
      take(lay->dphik, rows * D * 4);
      plan_phi_backward(pb, lay, &off);
    }
  } else {
    return fail(LUNA_ERR_INVALID_ARG, "unknown operation code");
  }
  lay->total = off;
  return LUNA_OK;
}

luna_status plan(const Problem& pb, Layout* lay, size_t room = SIZE_MAX) {
  return plan_within(room, lay, [&](Layout* l) { return plan_pieces(pb, l); });
}

luna_status check_ws(const Layout& lay, void* ws, size_t ws_bytes) {
  if (ws_bytes < lay.total) {
    char buf[128];
    snprintf(buf, sizeof buf, "workspace too small: need %zu bytes, got %zu", lay.total, ws_bytes);
    return fail(LUNA_ERR_WORKSPACE, buf);
  }
  if (ws == nullptr) return fail(LUNA_ERR_INVALID_ARG, "workspace is NULL");
  if (((uintptr_t)ws & 255) != 0) return fail(LUNA_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
  return LUNA_OK;
}

luna_status hip_fail(hipError_t e, const char* what) {
  return fail(LUNA_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

luna_status enqueue_prepare(const Problem& pb, uint8_t* ws, const Layout& lay, hipStream_t s) {
  const luna_phi_params* p = pb.p;
  luna::PrepareArgs a{};
  a.fc1_w = p->fc1_w;
  a.fc1_b = p->fc1_b;
  a.fc2_w = p->fc2_w;
  a.fc2_b = p->fc2_b;
  a.P = param_sets(pb);
  a.C1 = p->shared_channels ? 1 : p->L;
  a.L = p->L;
  a.hidden = p->hidden;
  a.M = p->M;
  a.nonneg = p->nonneg;
  a.tables = ws + lay.tables;
  hipError_t e = luna::launch_prepare(a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "table kernel launch");
}

luna::PhiArgs phi_args(const Problem& pb, uint8_t* ws, const Layout& lay) {
  luna::PhiArgs f{};
  f.W = pb.p->W;
  f.b = pb.p->b;
  f.tables = ws + lay.tables;
  f.M = pb.p->M;
  f.per_head = pb.p->per_head;
  return f;
}

bool finite_nonneg(float x) { return std::isfinite(x) && x >= 0.0f; }

// C (+)= A B (fp32) over (head, chunk) batches; strides of (head, chunk, row, column)
// for each operand; m/n/k_chunk: that dimension is the chunk's (ragged last chunk);
// lower: only the lower triangle of C (with the diagonal) is formed.
struct ChunkGemm {
  int heads, chunks, chunk, seq;
  hipStream_t s;
  hipError_t operator()(const float* A, int64_t ah, int64_t ac, int64_t ai, int64_t ak, const float* Bm, int64_t bh,
                        int64_t bc, int64_t bk, int64_t bj, float* Cm, int64_t ch, int64_t c2, int64_t ci, int64_t cj,
                        int Mm, int Nn, int Kk, int mc, int nc, int kc, int lower, int acc) const {
    luna::BwdGemm g{};
    g.A = A; g.sAh = ah; g.sAc = ac; g.sAi = ai; g.sAk = ak;
    g.B = Bm; g.sBh = bh; g.sBc = bc; g.sBk = bk; g.sBj = bj;
    g.C = Cm; g.sCh = ch; g.sCc = c2; g.sCi = ci; g.sCj = cj;
    g.M = Mm; g.N = Nn; g.K = Kk;
    g.heads = heads; g.chunks = chunks; g.chunk = chunk; g.seq = seq;
    g.m_chunk = mc; g.n_chunk = nc; g.k_chunk = kc; g.lower = lower; g.accumulate = acc;
    return luna::launch_bwd_gemm(g, s);
  }
};

// The attention part of the fp32 forward for given fp32 features (eq. (9) of
// Section 3.1, the causal form in 64-token chunks): [V | 1], per-chunk [S_c | z_c] =
// phi(K_c)^T [V_c | 1], their exclusive prefix over chunks (causal) or total, and with
// queries [num | den - eps] = phi(Q_c) [S_c | z_c] (+ P_c [V_c | 1], P_c =
// tril(phi(Q_c) phi(K_c)^T)).  phiq == nullptr: the state only.
luna_status enqueue_f32_attention(luna::Dt vdt, int64_t heads64, int64_t n, int dd, int D, uint8_t* w,
                                  const Layout& lay, const float* phiq, const float* phik, const void* V, bool causal,
                                  hipStream_t s) {
  const int heads = (int)heads64, E = dd + 1, C = lay.chunk, nch = lay.nch;
  const int64_t nD = n * D, nE = n * E, st_el = (int64_t)D * E, cc = (int64_t)C * C;
  float* vx = reinterpret_cast<float*>(w + lay.vx);
  float* y = reinterpret_cast<float*>(w + lay.y);
  float* sx = reinterpret_cast<float*>(w + lay.sx);
  float* pm = reinterpret_cast<float*>(w + lay.pm);
  hipError_t e;
#define LUNA_TRY(expr, what) \
  if ((e = (expr)) != hipSuccess) return hip_fail(e, what)
  LUNA_TRY(luna::launch_bwd_pack(vdt, V, vx, heads64 * n, dd, s), "pack kernel launch");
  const ChunkGemm gemm{heads, nch, C, (int)n, s};
  const int64_t sh = (int64_t)nch * st_el;  // head stride of the per-chunk states
  LUNA_TRY(gemm(phik, nD, (int64_t)C * D, 1, D, vx, nE, (int64_t)C * E, E, 1, sx, sh, st_el, E, 1, D, E, C, 0, 0, 1,
                0, 0), "state GEMM");
  LUNA_TRY(luna::launch_bwd_scan(sx, heads, nch, st_el, !causal, s), "state scan");
  if (!phiq) return LUNA_OK;
  LUNA_TRY(gemm(phiq, nD, (int64_t)C * D, D, 1, sx, sh, st_el, E, 1, y, nE, (int64_t)C * E, E, 1, C, E, D, 1, 0, 0,
                0, 0), "readout GEMM");
  if (causal) {
    LUNA_TRY(gemm(phiq, nD, (int64_t)C * D, D, 1, phik, nD, (int64_t)C * D, 1, D, pm, nch * cc, cc, C, 1, C, C, D, 1,
                  1, 0, 1, 0), "P GEMM");
    LUNA_TRY(gemm(pm, nch * cc, cc, C, 1, vx, nE, (int64_t)C * E, E, 1, y, nE, (int64_t)C * E, E, 1, C, E, C, 1, 0,
                  1, 0, 1), "intra-chunk GEMM");
  }
#undef LUNA_TRY
  return LUNA_OK;
}

// Features of the keys (and queries) in fp32 into the workspace.  Q == nullptr: keys only.
luna_status enqueue_f32_features(const Problem& pb, uint8_t* w, const Layout& lay, const void* Q, const void* K,
                                 hipStream_t s) {
  luna::FeatureMapArgs f{};  // queries and keys in one launch
  f.phi = phi_args(pb, w, lay);
  f.rows_per_head = pb.n;
  f.H = (int)pb.H;
  f.heads = pb.B * pb.H;
  f.X = K;
  f.out = w + lay.phik;
  if (Q) {
    f.X2 = Q;
    f.out2 = w + lay.phiq;
  }
  const hipError_t e = luna::launch_featuremap(pb.dt == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, luna::Dt::F32,
                                               (int)pb.d, pb.p->L, f, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "feature-map kernel launch");
}

// The non-causal attention from features in memory (eq. (9) of Section 3.1): statistics
// per piece, their total, and with queries the readout.
luna_status enqueue_feat_attention(luna::Dt fdt, luna::Dt vdt, int64_t heads, int64_t n, int d, int D, uint8_t* w,
                                   const Layout& lay, const void* phiq, const void* phik, const void* V, float eps,
                                   void* out, luna::FeatArgs* args, hipStream_t s) {
  luna::FeatArgs& a = *args;
  a.phiq = phiq;
  a.phik = phik;
  a.v = V;
  a.out = out;
  a.state = reinterpret_cast<float*>(w + lay.sx);
  a.heads = heads;
  a.n = n;
  a.elems = luna::feat_elems(d, D);
  a.D = D;
  a.piece = lay.chunk;
  a.pieces = lay.nch;
  a.eps = eps;
  hipError_t e = luna::launch_feat_state(fdt, vdt, d, a, s);
  if (e != hipSuccess) return hip_fail(e, "state kernel launch");
  if ((e = luna::launch_feat_total(a, s)) != hipSuccess) return hip_fail(e, "state sum launch");
  if (!phiq) return LUNA_OK;
  e = luna::launch_feat_readout(fdt, vdt, d, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "readout kernel launch");
}

// Arguments of the chunk kernels: statistics at `state`, rows x with values u, columns y
// with values v.
luna::ChunkArgs chunk_args(int64_t heads, int64_t n, int d, int D, const Layout& lay, bool causal, const float* x,
                           const void* u, const float* y, const void* v, const float* state, float eps) {
  luna::ChunkArgs a{};
  a.x = x;
  a.u = u;
  a.y = y;
  a.v = v;
  a.state = state;
  a.heads = heads;
  a.n = n;
  a.elems = luna::feat_elems(d, D);
  a.D = D;
  a.piece = lay.chunk;
  a.pieces = lay.nch;
  a.causal = causal;
  a.eps = eps;
  return a;
}

// Statistics of every piece (weighted by w when given) into `state`, then what the chunk
// kernels start from: the exclusive prefix (suffix) over pieces, or the total.
luna_status enqueue_chunk_state(luna::Dt vdt, int64_t heads, int64_t n, int d, int D, const Layout& lay, bool causal,
                                bool suffix, const float* phi, const void* V, const float* wt, float* state,
                                hipStream_t s) {
  luna::FeatArgs a{};
  a.phik = phi;
  a.v = V;
  a.w = wt;
  a.state = state;
  a.heads = heads;
  a.n = n;
  a.elems = luna::feat_elems(d, D);
  a.D = D;
  a.piece = lay.chunk;
  a.pieces = lay.nch;
  hipError_t e = luna::launch_feat_state(luna::Dt::F32, vdt, d, a, s);
  if (e != hipSuccess) return hip_fail(e, "state kernel launch");
  e = causal ? luna::launch_chunk_scan(state, heads, lay.nch, a.elems, suffix, s) : luna::launch_feat_total(a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "state scan launch");
}

// The causal forward from given fp32 features: out = num / den in the value type.
luna_status enqueue_f32_causal(luna::Dt vdt, int64_t heads, int64_t n, int d, int D, uint8_t* w, const Layout& lay,
                               const float* phiq, const float* phik, const void* V, float eps, void* out,
                               hipStream_t s) {
  hipError_t e;
  if (!lay.chunked) {
    const luna_status st = enqueue_f32_attention(vdt, heads, n, d, D, w, lay, phiq, phik, V, true, s);
    if (st != LUNA_OK) return st;
    e = luna::launch_fwd_out(vdt, reinterpret_cast<const float*>(w + lay.y), out, heads * n, d, eps, s);
    return e == hipSuccess ? LUNA_OK : hip_fail(e, "output kernel launch");
  }
  float* state = reinterpret_cast<float*>(w + lay.sx);
  const luna_status st = enqueue_chunk_state(vdt, heads, n, d, D, lay, true, false, phik, V, nullptr, state, s);
  if (st != LUNA_OK) return st;
  luna::ChunkArgs a = chunk_args(heads, n, d, D, lay, true, phiq, nullptr, phik, V, state, eps);
  a.out = out;
  e = luna::launch_chunk_query(vdt, d, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "chunk kernel launch");
}

// The generic forward: the features in fp32, then attention from them.
luna_status enqueue_generic_attn(const Problem& pb, uint8_t* w, const Layout& lay, const void* Q, const void* K,
                                 const void* V, float eps, void* out, bool causal, hipStream_t s) {
  const luna_status st = enqueue_f32_features(pb, w, lay, Q, K, s);
  if (st != LUNA_OK) return st;
  const luna::Dt dt = pb.dt == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  const int64_t heads = pb.B * pb.H;
  const int D = pb.p->M * pb.p->L, d = (int)pb.d;
  const float* phiq = reinterpret_cast<const float*>(w + lay.phiq);
  const float* phik = reinterpret_cast<const float*>(w + lay.phik);
  if (causal) return enqueue_f32_causal(dt, heads, pb.n, d, D, w, lay, phiq, phik, V, eps, out, s);
  luna::FeatArgs a{};
  return enqueue_feat_attention(luna::Dt::F32, dt, heads, pb.n, d, D, w, lay, phiq, phik, V, eps, out, &a, s);
}

// Scratch of luna_attn_fwd_causal_noalloc: one array per device, part of the code
// object, so that calls need no allocation.  Host code never uses the array's name as
// an address (on the host it only stands in for the symbol): the device address comes
// from hipGetSymbolAddress, once per device, and is kept here.
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) uint8_t scratch[kScratchBytes];
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch.
luna_status scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(LUNA_ERR_UNSUPPORTED, "device index must be below 64");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress of the scratch array");
    if (ptr == nullptr || ((uintptr_t)ptr & 255) != 0) return fail(LUNA_ERR_HIP, "scratch array address not 256-byte aligned");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return LUNA_OK;
}

// A variant description's features per row (D) after checking it completely.
luna_status check_variant(const luna_phi_variant* v, int64_t* D) {
  if (v == nullptr || v->base == nullptr) return fail(LUNA_ERR_INVALID_ARG, "variant or its base parameters is NULL");
  const luna_phi_params* p = v->base;
  if (v->kind < LUNA_PHI_MLP || v->kind > LUNA_PHI_PERFORMER) return fail(LUNA_ERR_INVALID_ARG, "unknown variant kind");
  if (p->M < 1 || p->M > 256) return fail(LUNA_ERR_INVALID_ARG, "M must be in [1, 256]");
  if (p->per_head != 0 && p->per_head != 1) return fail(LUNA_ERR_INVALID_ARG, "per_head must be 0 or 1");
  if (!p->W || !p->b) return fail(LUNA_ERR_INVALID_ARG, "W or b is NULL");
  if ((v->env_w == nullptr) != (v->env_b == nullptr)) return fail(LUNA_ERR_INVALID_ARG, "env_w and env_b go together");
  if (v->ch_rms != 0 && v->ch_rms != 1) return fail(LUNA_ERR_INVALID_ARG, "ch_rms must be 0 or 1");
  if (v->kind != LUNA_PHI_MLP) {
    if (v->env_w || v->bank || v->ch_rms)
      return fail(LUNA_ERR_INVALID_ARG, "an envelope, bank or channel RMS needs the channel-MLP kind");
    *D = v->kind == LUNA_PHI_RFF_SINCOS ? 2 * (int64_t)p->M : p->M;
    return LUNA_OK;
  }
  if (v->act < LUNA_ACT_RELU || v->act > LUNA_ACT_TANH) return fail(LUNA_ERR_INVALID_ARG, "unknown activation");
  if (p->L < 1 || p->L > 16) return fail(LUNA_ERR_INVALID_ARG, "L must be in [1, 16]");
  if (p->hidden < 1 || p->hidden > 64) return fail(LUNA_ERR_INVALID_ARG, "hidden must be in [1, 64]");
  if (p->shared_channels != 0 && p->shared_channels != 1) return fail(LUNA_ERR_INVALID_ARG, "shared_channels must be 0 or 1");
  if (p->nonneg != 0 && p->nonneg != 1) return fail(LUNA_ERR_INVALID_ARG, "nonneg must be 0 or 1");
  if (!p->fc1_w || !p->fc1_b || !p->fc2_w || !p->fc2_b) return fail(LUNA_ERR_INVALID_ARG, "a channel-MLP array is NULL");
  if (v->ch_rms && !(std::isfinite(v->ch_rms_target) && v->ch_rms_target > 0.0f))
    return fail(LUNA_ERR_INVALID_ARG, "ch_rms_target must be finite and > 0");
  *D = v->bank ? (int64_t)p->M : (int64_t)p->M * p->L;
  if (*D > 512) return fail(LUNA_ERR_INVALID_ARG, "a variant has at most 512 features");
  return LUNA_OK;
}

// Workspace of a variant map of `rows` rows: with channel RMS, the per-workgroup
// partial sums, the channel scales and y of every row in fp32 ([row][M][L]).
constexpr size_t kVarPartialBytes = (size_t)luna::kVariantMaxGrid * luna::kVariantMaxL * sizeof(double);
constexpr size_t kVarScaleBytes = 256;
size_t variant_ws_bytes(const luna_phi_variant* v, int64_t rows) {
  if (v->kind != LUNA_PHI_MLP || !v->ch_rms) return 0;
  return align256(kVarPartialBytes) + kVarScaleBytes +
         align256((size_t)rows * (size_t)v->base->M * (size_t)v->base->L * sizeof(float));
}

// Buffers of luna_attn_fwd_features: the causal scan kernel on the bf16 features when
// it is built for (d, D), non-causal the kernels on features in their own type, else the
// fp32 path (fp32 copies of bf16 features).
luna_status plan_features_pieces(luna_dtype phi_dtype, luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                                 int64_t D, int32_t causal, int32_t chunk, Layout* lay) {
  if ((phi_dtype != LUNA_F32 && phi_dtype != LUNA_BF16) || (dtype != LUNA_F32 && dtype != LUNA_BF16))
    return fail(LUNA_ERR_INVALID_ARG, "dtypes must be LUNA_F32 or LUNA_BF16");
  if (B < 1 || H < 1 || n < 1) return fail(LUNA_ERR_INVALID_ARG, "B, H and n must be >= 1");
  if (n > (int64_t)1 << 30 || B * H > (int64_t)1 << 24) return fail(LUNA_ERR_UNSUPPORTED, "n or B*H too large");
  if (d < 1 || d > 256) return fail(LUNA_ERR_UNSUPPORTED, "d must be in [1, 256]");
  if (D < 1 || D > 512) return fail(LUNA_ERR_UNSUPPORTED, "D must be in [1, 512]");
  if (causal != 0 && causal != 1) return fail(LUNA_ERR_INVALID_ARG, "causal must be 0 or 1");
  if (causal && chunk != 64) return fail(LUNA_ERR_UNSUPPORTED, "chunk must be 64");
  const int64_t heads = B * H;
  const luna::Dt vdt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  size_t off = 0;
  if (causal && phi_dtype == LUNA_BF16 && dtype == LUNA_BF16 && luna::causal_given_supported(luna::Dt::BF16, (int)d, (int)D)) {
    lay->given = 1;
    plan_causal_parts(luna::Dt::BF16, heads, n, luna::causal_given_state_floats((int)d, (int)D), lay, &off, false);
  } else if (!causal && luna::feat_supported((int)d, (int)D)) {
    // the features in their own type: statistics of pieces only
    lay->feat = 1;
    if ((n + 511) / 512 > 65535) return fail(LUNA_ERR_UNSUPPORTED, "n must be <= 65535 * 512");
    lay->chunk = state_piece(phi_dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, vdt, heads, n, (int)d, (int)D,
                             lay->few);
    const int64_t pieces = (n + lay->chunk - 1) / lay->chunk;
    lay->nch = (int)pieces;
    lay->sx = off;
    off = align256(off + (size_t)heads * lay->nch * (size_t)luna::feat_elems(d, D) * 4);
  } else {
    lay->generic = 1;
    luna_status st =
        plan_f32_buffers(vdt, heads, n, (int)d, (int)D, causal != 0, true, phi_dtype == LUNA_BF16, lay, &off);
    if (st != LUNA_OK) return st;
  }
  lay->total = off;
  return LUNA_OK;
}

luna_status plan_features(luna_dtype phi_dtype, luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                          int64_t D, int32_t causal, int32_t chunk, Layout* lay, size_t room = SIZE_MAX) {
  return plan_within(room, lay, [&](Layout* l) {
    return plan_features_pieces(phi_dtype, dtype, B, H, n, d, D, causal, chunk, l);
  });
}

// The causal kernel over its parts: with more than one, the state launch first (and the
// running sums of equal parts' states).  `launch` launches the kernel with `a`.
template <typename Launch>
luna_status enqueue_causal_parts(const Layout& lay, uint8_t* w, luna::CausalArgs& a, Launch launch, hipStream_t s) {
  hipError_t e;
  if (lay.parts > 1) {
    float* st = reinterpret_cast<float*>(w + lay.state);
    a.pieces = lay.pieces;
    a.piece_chunks = lay.piece_chunks;
    a.part_chunks = lay.part_chunks;
    a.state_out = st;
    if ((e = launch()) != hipSuccess) return hip_fail(e, "causal attention state launch");
    if (lay.part_chunks) {
      e = luna::launch_causal_prefix(st, a.heads, lay.pieces, lay.state_floats, s);
      if (e != hipSuccess) return hip_fail(e, "causal state sum launch");
    }
    a.state_out = nullptr;
    a.state_in = st;
  }
  e = launch();
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "causal attention kernel launch");
}

// Through the feature map, from dphi(Q) and dphi(K) in the workspace (fp32, [head][n][D]):
// dx into dQ, dK (when given), [dW | db] and the channel-MLP gradients into grads (when
// given).  Used by the backward pass and by the distillation loss.
luna_status enqueue_phi_backward(const Problem& pb, uint8_t* w, const Layout& lay, const void* Q, const void* K,
                                 void* dQ, void* dK, const luna_phi_grads* grads, hipStream_t s) {
  const luna_phi_params* p = pb.p;
  const int M = p->M, L = p->L, dd = (int)pb.d, P = param_sets(pb);
  hipError_t e;
#define LUNA_TRY(expr, what) \
  if ((e = (expr)) != hipSuccess) return hip_fail(e, what)
  luna::MapBwd a{};
  a.xq = Q;
  a.xk = K;
  a.dphiq = reinterpret_cast<const float*>(w + lay.dphiq);
  a.dphik = reinterpret_cast<const float*>(w + lay.dphik);
  a.dxq = dQ;
  a.dxk = dK;
  if (grads) {
    a.duq = reinterpret_cast<float*>(w + lay.duq);
    a.duk = reinterpret_cast<float*>(w + lay.duk);
  }
  a.W = p->W;
  a.b = p->b;
  a.tables = w + lay.tables;
  a.partial = reinterpret_cast<float*>(w + lay.bpart);
  a.dw_partial = reinterpret_cast<float*>(w + lay.dwp);
  a.n = pb.n;
  a.heads = pb.B * pb.H;
  a.H = (int)pb.H;
  a.M = M;
  a.per_head = p->per_head;
  a.groups = lay.groups;
  a.dw_groups = lay.dw_groups;
  a.part_floats = lay.part_floats;
  LUNA_TRY(luna::launch_map_bwd(pb.dt == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, dd, L, a, P, s),
           "feature-map backward kernel launch");
  if (grads) {
    LUNA_TRY(luna::launch_bwd_dw(a.dw_partial, grads->W, grads->b, lay.dw_groups, M, dd, P, s), "weight-gradient sum");
    const int units = (p->shared_channels ? 1 : L) * p->hidden;
    const int used = 2 * (units + 1) * L;
    double* sum = reinterpret_cast<double*>(w + lay.sum);
    double* pre = reinterpret_cast<double*>(w + lay.pre);
    LUNA_TRY(luna::launch_bwd_reduce(a.partial, sum, lay.groups, lay.part_floats, used, P, s), "reduce kernel launch");
    LUNA_TRY(luna::launch_bwd_prefix(sum, pre, w + lay.tables, M, dd, L, lay.part_floats, luna::bwd_nseg_cap(L), P, s),
             "prefix kernel launch");
    luna::BwdMlp m{};
    m.sum = sum;
    m.pre = pre;
    m.tables = w + lay.tables;
    m.fc1_w = p->fc1_w;
    m.fc1_b = p->fc1_b;
    m.fc2_w = p->fc2_w;
    m.dfc1_w = grads->fc1_w;
    m.dfc1_b = grads->fc1_b;
    m.dfc2_w = grads->fc2_w;
    m.dfc2_b = grads->fc2_b;
    m.L = L;
    m.hidden = p->hidden;
    m.C1 = p->shared_channels ? 1 : L;
    m.part_floats = lay.part_floats;
    m.nseg_cap = luna::bwd_nseg_cap(L);
    LUNA_TRY(luna::launch_bwd_mlp(m, P, s), "parameter-gradient kernel launch");
  }
#undef LUNA_TRY
  return LUNA_OK;
}

}  // namespace

extern "C" {

int64_t luna_phi_variant_features(const luna_phi_variant* v) {
  int64_t D = -1;
  return check_variant(v, &D) == LUNA_OK ? D : -1;
}

size_t luna_featuremap_variant_workspace_bytes(luna_dtype, int64_t B, int64_t H, int64_t n, int64_t,
                                               const luna_phi_variant* v) {
  int64_t D = 0;
  if (B < 1 || H < 1 || n < 1 || n > (int64_t)1 << 30 || B * H > (int64_t)1 << 24) return 0;
  return check_variant(v, &D) == LUNA_OK ? variant_ws_bytes(v, B * H * n) : 0;
}

luna_status luna_featuremap_variant(const void* X, luna_dtype x_dtype, int64_t B, int64_t H, int64_t n,
                                    int64_t d, const luna_phi_variant* v, void* phi_out, luna_dtype out_dtype,
                                    void* ws, size_t ws_bytes, void* stream) {
  g_last_error.clear();
  int64_t D = 0;
  luna_status st = check_variant(v, &D);
  if (st != LUNA_OK) return st;
  if ((x_dtype != LUNA_F32 && x_dtype != LUNA_BF16) || (out_dtype != LUNA_F32 && out_dtype != LUNA_BF16))
    return fail(LUNA_ERR_INVALID_ARG, "dtypes must be LUNA_F32 or LUNA_BF16");
  if (B < 1 || H < 1 || n < 1) return fail(LUNA_ERR_INVALID_ARG, "B, H and n must be >= 1");
  if (n > (int64_t)1 << 30 || B * H > (int64_t)1 << 24) return fail(LUNA_ERR_UNSUPPORTED, "n or B*H too large");
  if (d != 32 && d != 64 && d != 128) return fail(LUNA_ERR_UNSUPPORTED, "d must be 32, 64 or 128");
  if (!X || !phi_out) return fail(LUNA_ERR_INVALID_ARG, "X or phi_out is NULL");
  const size_t need = variant_ws_bytes(v, B * H * n);
  if (need) {
    Layout lay;
    lay.total = need;
    if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  }
  const luna_phi_params* p = v->base;
  luna::VariantArgs a{};
  a.X = X;
  a.out = phi_out;
  a.W = p->W;
  a.b = p->b;
  a.kind = v->kind;
  a.M = p->M;
  a.per_head = p->per_head;
  a.H = (int)H;
  a.rows_per_head = n;
  a.heads = B * H;
  a.L = 1;
  a.hidden = 1;
  a.C1 = 1;
  if (v->kind == LUNA_PHI_MLP) {
    a.act = v->act;
    a.L = p->L;
    a.hidden = p->hidden;
    a.C1 = p->shared_channels ? 1 : p->L;
    a.nonneg = p->nonneg;
    a.fc1_w = p->fc1_w;
    a.fc1_b = p->fc1_b;
    a.fc2_w = p->fc2_w;
    a.fc2_b = p->fc2_b;
    a.env_w = v->env_w;
    a.env_b = v->env_b;
    a.bank = v->bank;
  }
  const luna::Dt idt = x_dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  a.out_bf16 = out_dtype == LUNA_BF16;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e;
  int grid = 0;
  if (need) {  // channel RMS: y and the sums of y^2, the scales, then phi from y
    uint8_t* w = static_cast<uint8_t*>(ws);
    double* partial = reinterpret_cast<double*>(w);
    float* scale = reinterpret_cast<float*>(w + align256(kVarPartialBytes));
    a.rms_pass = 1;
    a.rms_partial = partial;
    a.rms_y = reinterpret_cast<float*>(w + align256(kVarPartialBytes) + kVarScaleBytes);
    if ((e = luna::launch_variant_map(idt, (int)d, a, &grid, s)) != hipSuccess) return hip_fail(e, "variant map launch");
    const double count = (double)(B * H) * (double)n * (double)p->M;
    if ((e = luna::launch_variant_rms(partial, grid, p->L, count, v->ch_rms_target, scale, s)) != hipSuccess)
      return hip_fail(e, "channel RMS kernel launch");
    e = luna::launch_variant_finish(a, scale, s);
    return e == hipSuccess ? LUNA_OK : hip_fail(e, "channel RMS output kernel launch");
  }
  e = luna::launch_variant_map(idt, (int)d, a, &grid, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "variant map launch");
}

size_t luna_attn_features_workspace_bytes(luna_dtype phi_dtype, luna_dtype dtype, int64_t B, int64_t H, int64_t n,
                                          int64_t d, int64_t D, int32_t causal, int32_t chunk) {
  Layout lay;
  return plan_features(phi_dtype, dtype, B, H, n, d, D, causal, chunk, &lay) == LUNA_OK ? lay.total : 0;
}

luna_status luna_attn_fwd_features(const void* phiQ, const void* phiK, luna_dtype phi_dtype, const void* V,
                                   luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d, int64_t D,
                                   int32_t causal, int32_t chunk, float eps, void* out, void* ws, size_t ws_bytes,
                                   void* stream) {
  g_last_error.clear();
  Layout lay;
  luna_status st = plan_features(phi_dtype, dtype, B, H, n, d, D, causal, chunk, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!phiQ || !phiK || !V || !out) return fail(LUNA_ERR_INVALID_ARG, "phiQ, phiK, V or out is NULL");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if (lay.total && (st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  const luna::Dt vdt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  hipError_t e;
  if (lay.given) {  // the causal scan kernel on the bf16 features
    luna::CausalArgs a{};
    a.Q = phiQ;
    a.K = phiK;
    a.V = V;
    a.out = out;
    a.phi.M = (int)D;
    a.n = (int)n;
    a.H = (int)H;
    a.heads = (int)(B * H);
    a.parts = lay.parts;
    a.split = lay.split;
    a.eps = eps;
    a.phiq = phiQ;
    a.phik = phiK;
    return enqueue_causal_parts(lay, w, a, [&]() { return luna::launch_causal_given((int)d, (int)D, a, s); }, s);
  }
  const int64_t heads = B * H;
  if (lay.feat) {
    luna::FeatArgs a{};
    return enqueue_feat_attention(phi_dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, vdt, heads, n, (int)d, (int)D,
                                  w, lay, phiQ, phiK, V, eps, out, &a, s);
  }
  const float* fq = static_cast<const float*>(phiQ);
  const float* fk = static_cast<const float*>(phiK);
  if (phi_dtype == LUNA_BF16) {  // fp32 copies of the features
    float* q32 = reinterpret_cast<float*>(w + lay.phiq);
    float* k32 = reinterpret_cast<float*>(w + lay.phik);
    if ((e = luna::launch_widen(luna::Dt::BF16, phiQ, q32, heads * n * D, s)) != hipSuccess) return hip_fail(e, "widen");
    if ((e = luna::launch_widen(luna::Dt::BF16, phiK, k32, heads * n * D, s)) != hipSuccess) return hip_fail(e, "widen");
    fq = q32;
    fk = k32;
  }
  if (causal) return enqueue_f32_causal(vdt, heads, n, (int)d, (int)D, w, lay, fq, fk, V, eps, out, s);
  if ((st = enqueue_f32_attention(vdt, heads, n, (int)d, (int)D, w, lay, fq, fk, V, false, s)) != LUNA_OK) return st;
  e = luna::launch_fwd_out(vdt, reinterpret_cast<const float*>(w + lay.y), out, heads * n, (int)d, eps, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "output kernel launch");
}


size_t luna_workspace_bytes(int32_t op, luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                            const luna_phi_params* p, int32_t chunk) {
  Problem pb{op, dtype, B, H, n, d, p, chunk};
  Layout lay;
  return plan(pb, &lay) == LUNA_OK ? lay.total : 0;
}

luna_status luna_featuremap(const void* X, luna_dtype x_dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                            const luna_phi_params* p, void* phi_out, luna_dtype out_dtype, void* ws,
                            size_t ws_bytes, void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_FEATUREMAP, x_dtype, B, H, n, d, p, 0};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (out_dtype != LUNA_F32 && out_dtype != LUNA_BF16) return fail(LUNA_ERR_INVALID_ARG, "out_dtype must be LUNA_F32 or LUNA_BF16");
  if (!X || !phi_out) return fail(LUNA_ERR_INVALID_ARG, "X or phi_out is NULL");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  luna::FeatureMapArgs a{};
  a.X = X;
  a.out = phi_out;
  a.phi = phi_args(pb, w, lay);
  a.rows_per_head = n;
  a.H = (int)H;
  a.heads = B * H;
  hipError_t e = luna::launch_featuremap(x_dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32,
                                         out_dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, (int)d, p->L, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "feature-map kernel launch");
}

luna_status luna_attn_fwd(const void* Q, const void* K, const void* V, luna_dtype dtype, int64_t B, int64_t H,
                          int64_t n, int64_t d, const luna_phi_params* p, float eps, void* out, void* ws,
                          size_t ws_bytes, void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_ATTN, dtype, B, H, n, d, p, 0};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!Q || !K || !V || !out) return fail(LUNA_ERR_INVALID_ARG, "Q, K, V or out is NULL");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  if (lay.generic) return enqueue_generic_attn(pb, w, lay, Q, K, V, eps, out, false, s);
  luna::NoncausalArgs a{};
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.out = out;
  a.phi = phi_args(pb, w, lay);
  a.n = (int)n;
  a.H = (int)H;
  a.heads = (int)(B * H);
  a.splits = lay.splits;
  a.tokens_per_split = lay.tokens_per_split;
  a.eps = eps;
  a.partial = reinterpret_cast<float*>(w + lay.partial);
  a.frags = w + lay.frags;
  a.tile_tokens = lay.tile_tokens;
  a.tiles = lay.tiles;
  a.fused = lay.fused;
  hipError_t e = luna::launch_noncausal(dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32, (int)d, p->L, p->M, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "attention kernel launch");
}

luna_status luna_attn_fwd_causal(const void* Q, const void* K, const void* V, luna_dtype dtype, int64_t B,
                                 int64_t H, int64_t n, int64_t d, const luna_phi_params* p, int32_t chunk, float eps,
                                 void* out, void* ws, size_t ws_bytes, void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_ATTN_CAUSAL, dtype, B, H, n, d, p, chunk};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!Q || !K || !V || !out) return fail(LUNA_ERR_INVALID_ARG, "Q, K, V or out is NULL");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  if (lay.generic) return enqueue_generic_attn(pb, w, lay, Q, K, V, eps, out, true, s);
  luna::CausalArgs a{};
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.out = out;
  a.phi = phi_args(pb, w, lay);
  a.n = (int)n;
  a.H = (int)H;
  a.heads = (int)(B * H);
  a.parts = lay.parts;
  a.split = lay.split;
  a.eps = eps;
  const luna::Dt dt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  const int D = p->M * p->L;
  if (lay.given) {  // phi(Q), phi(K) in bf16 first (one launch)
    luna::FeatureMapArgs f{};
    f.phi = a.phi;
    f.rows_per_head = n;
    f.H = (int)H;
    f.heads = B * H;
    f.X = Q;
    f.out = w + lay.phiq;
    f.X2 = K;
    f.out2 = w + lay.phik;
    hipError_t e = luna::launch_featuremap(dt, luna::Dt::BF16, (int)d, p->L, f, s);
    if (e != hipSuccess) return hip_fail(e, "feature-map kernel launch");
    a.phiq = w + lay.phiq;
    a.phik = w + lay.phik;
  }
  auto launch = [&]() {
    return lay.given ? luna::launch_causal_given((int)d, D, a, s) : luna::launch_causal(dt, (int)d, p->L, p->M, a, s);
  };
  if (lay.staged) {
    // launch 1: part 0 scans [0, A), part 1 sums the state of [A, A + B); both write
    // their final states as pieces 0 and 1.  launch 2: part 0 scans [A, A + B) from
    // piece 0, part 1 scans [A + B, nch) from pieces 0 + 1.
    const int A = lay.sa, AB = lay.sa + lay.sb, nch = (int)((n + 63) / 64);
    float* st = reinterpret_cast<float*>(w + lay.state);
    a.staged = 1;
    a.pieces = 2;
    a.pc_first[0] = 0;  a.pc_begin[0] = 0;  a.pc_end[0] = A;  a.pseed[0] = 0;
    a.pc_first[1] = A;  a.pc_begin[1] = AB; a.pc_end[1] = AB; a.pseed[1] = 0;
    a.state_fin = st;
    hipError_t e = launch();
    if (e != hipSuccess) return hip_fail(e, "causal attention first scan launch");
    a.pc_first[0] = A;  a.pc_begin[0] = A;  a.pc_end[0] = AB;  a.pseed[0] = 1;
    a.pc_first[1] = AB; a.pc_begin[1] = AB; a.pc_end[1] = nch; a.pseed[1] = 2;
    a.state_fin = nullptr;
    a.state_in = st;
    e = launch();
    return e == hipSuccess ? LUNA_OK : hip_fail(e, "causal attention second scan launch");
  }
  return enqueue_causal_parts(lay, w, a, launch, s);
}

luna_status luna_attn_fwd_causal_noalloc(const void* Q, const void* K, const void* V, luna_dtype dtype,
                                         int64_t B, int64_t H, int64_t n, int64_t d, const luna_phi_params* p,
                                         int32_t chunk, float eps, void* out, void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_ATTN_CAUSAL, dtype, B, H, n, d, p, chunk};
  Layout lay;
  luna_status st = plan(pb, &lay, kScratchBytes);
  if (st != LUNA_OK) return st;
  if (lay.total > kScratchBytes) {
    char buf[160];
    snprintf(buf, sizeof buf, "problem needs %zu bytes of scratch; the static scratch holds %zu", lay.total,
             kScratchBytes);
    return fail(LUNA_ERR_WORKSPACE, buf);
  }
  void* ws = nullptr;
  if ((st = scratch_address(&ws)) != LUNA_OK) return st;
  return luna_attn_fwd_causal(Q, K, V, dtype, B, H, n, d, p, chunk, eps, out, ws, kScratchBytes, stream);
}

size_t luna_noalloc_scratch_bytes(void) { return kScratchBytes; }

luna_status luna_attn_state(const void* K, const void* V, luna_dtype dtype, int64_t B, int64_t H, int64_t n,
                            int64_t d, const luna_phi_params* p, int32_t accumulate, float* S, float* z, void* ws,
                            size_t ws_bytes, void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_STATE, dtype, B, H, n, d, p, 0};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!K || !V || !S || !z) return fail(LUNA_ERR_INVALID_ARG, "K, V, S or z is NULL");
  if (accumulate != 0 && accumulate != 1) return fail(LUNA_ERR_INVALID_ARG, "accumulate must be 0 or 1");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  const luna::Dt dt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  if (lay.generic) {
    if ((st = enqueue_f32_features(pb, w, lay, nullptr, K, s)) != LUNA_OK) return st;
    luna::FeatArgs a{};
    st = enqueue_feat_attention(luna::Dt::F32, dt, B * H, n, (int)d, p->M * p->L, w, lay, nullptr, w + lay.phik, V, 0.0f,
                                nullptr, &a, s);
    if (st != LUNA_OK) return st;
    const hipError_t e = luna::launch_feat_export((int)d, a, S, z, accumulate, s);
    return e == hipSuccess ? LUNA_OK : hip_fail(e, "state export kernel launch");
  }
  if (lay.pieces == 0) {
    luna::NoncausalArgs a{};
    a.K = K;
    a.V = V;
    a.phi = phi_args(pb, w, lay);
    a.n = (int)n;
    a.H = (int)H;
    a.heads = (int)(B * H);
    a.splits = lay.splits;
    a.tokens_per_split = lay.tokens_per_split;
    a.partial = reinterpret_cast<float*>(w + lay.partial);
    a.state_S = S;
    a.state_z = z;
    a.accumulate = accumulate;
    hipError_t e = luna::launch_state(dt, (int)d, p->L, p->M, a, s);
    return e == hipSuccess ? LUNA_OK : hip_fail(e, "state kernel launch");
  }
  luna::CausalArgs a{};
  a.K = K;
  a.V = V;
  a.Q = K;  // (the state launch reads no query rows)
  a.phi = phi_args(pb, w, lay);
  a.n = (int)n;
  a.H = (int)H;
  a.heads = (int)(B * H);
  a.parts = 2;
  a.split = lay.split;
  a.pieces = lay.pieces;
  a.piece_chunks = lay.piece_chunks;
  a.state_out = reinterpret_cast<float*>(w + lay.state);
  hipError_t e = luna::launch_causal(dt, (int)d, p->L, p->M, a, s);
  if (e != hipSuccess) return hip_fail(e, "causal state launch");
  a.export_S = S;
  a.export_z = z;
  a.accumulate = accumulate;
  e = luna::launch_causal(dt, (int)d, p->L, p->M, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "state export launch");
}

luna_status luna_attn_causal_step(const void* Q, const void* K, const void* V, luna_dtype dtype, int64_t B,
                                  int64_t H, int64_t m, int64_t d, const luna_phi_params* p, float eps,
                                  int32_t tables_ready, float* S, float* z, void* out, void* ws, size_t ws_bytes,
                                  void* stream) {
  g_last_error.clear();
  Problem pb{LUNA_OP_CAUSAL_STEP, dtype, B, H, m, d, p, 0};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!Q || !K || !V || !S || !z || !out) return fail(LUNA_ERR_INVALID_ARG, "Q, K, V, S, z or out is NULL");
  if (((uintptr_t)S & 15) != 0) return fail(LUNA_ERR_INVALID_ARG, "S must be 16-byte aligned");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if (tables_ready != 0 && tables_ready != 1) return fail(LUNA_ERR_INVALID_ARG, "tables_ready must be 0 or 1");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if (!tables_ready && (st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  const luna::Dt dt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  luna::FeatureMapArgs f{};  // queries and keys in one launch
  f.phi = phi_args(pb, w, lay);
  f.rows_per_head = m;
  f.H = (int)H;
  f.heads = B * H;
  if (!p->per_head && B * H * m <= ((int64_t)1 << 30)) {
    // one parameter set: the rows of all heads are one contiguous array, mapped in
    // 64-row tiles across heads (a one-token step then needs B*H/64 tiles, not B*H)
    f.rows_per_head = B * H * m;
    f.H = 1;
    f.heads = 1;
  }
  f.X = Q;
  f.out = w + lay.phiq;
  f.X2 = K;
  f.out2 = w + lay.phik;
  // z before the step, for every column block of a head to read (block 0 rewrites z),
  // copied by workgroups of the same launch
  f.copy_src = z;
  f.copy_dst = reinterpret_cast<float*>(w + lay.zcopy);
  f.copy_n = (B * H) * (int64_t)(p->M * p->L);
  hipError_t e = luna::launch_featuremap(dt, luna::Dt::F32, (int)d, p->L, f, s);
  if (e != hipSuccess) return hip_fail(e, "feature-map kernel launch");
  luna::StepArgs a{};
  a.phiq = reinterpret_cast<const float*>(w + lay.phiq);
  a.phik = reinterpret_cast<const float*>(w + lay.phik);
  a.V = V;
  a.out = out;
  a.S = S;
  a.z = z;
  a.z_in = reinterpret_cast<const float*>(w + lay.zcopy);
  a.m = (int)m;
  a.d = (int)d;
  a.D = p->M * p->L;
  a.heads = (int)(B * H);
  a.eps = eps;
  e = luna::launch_causal_step(dt, a, s);
  return e == hipSuccess ? LUNA_OK : hip_fail(e, "streaming step kernel launch");
}

luna_status luna_attn_bwd(const void* Q, const void* K, const void* V, const void* dO, luna_dtype dtype, int64_t B,
                          int64_t H, int64_t n, int64_t d, const luna_phi_params* p, int32_t causal, float eps,
                          void* dQ, void* dK, void* dV, const luna_phi_grads* grads, void* ws, size_t ws_bytes,
                          void* stream) {
  g_last_error.clear();
  if (causal != 0 && causal != 1) return fail(LUNA_ERR_INVALID_ARG, "causal must be 0 or 1");
  Problem pb{causal ? LUNA_OP_ATTN_CAUSAL_BWD : LUNA_OP_ATTN_BWD, dtype, B, H, n, d, p, 64};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!Q || !K || !V || !dO || !dQ || !dK || !dV) return fail(LUNA_ERR_INVALID_ARG, "an input or output is NULL");
  if (grads && (!grads->W || !grads->b || !grads->fc1_w || !grads->fc1_b || !grads->fc2_w || !grads->fc2_b))
    return fail(LUNA_ERR_INVALID_ARG, "a parameter-gradient array is NULL");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  const luna::Dt dt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  const int D = p->M * p->L, dd = (int)d;
  const int64_t heads = B * H;
  const float* phiq = reinterpret_cast<const float*>(w + lay.phiq);
  const float* phik = reinterpret_cast<const float*>(w + lay.phik);
  float* sx = reinterpret_cast<float*>(w + lay.sx);
  float* dsx = reinterpret_cast<float*>(w + lay.dsx);
  float* wq = reinterpret_cast<float*>(w + lay.wq);
  if ((st = enqueue_f32_features(pb, w, lay, Q, K, s)) != LUNA_OK) return st;
  // [S | z]; 1 / den, dden and dphi(Q)
  if ((st = enqueue_chunk_state(dt, heads, n, dd, D, lay, causal, false, phik, V, nullptr, sx, s)) != LUNA_OK) return st;
  luna::ChunkArgs a = chunk_args(heads, n, dd, D, lay, causal, phiq, dO, phik, V, sx, eps);
  a.w = wq;
  a.dx = reinterpret_cast<float*>(w + lay.dphiq);
  hipError_t e = luna::launch_chunk_query(dt, dd, a, s);
  if (e != hipSuccess) return hip_fail(e, "query-gradient kernel launch");
  // [dS | dz]; dphi(K) and dV
  if ((st = enqueue_chunk_state(dt, heads, n, dd, D, lay, causal, true, phiq, dO, wq, dsx, s)) != LUNA_OK) return st;
  a = chunk_args(heads, n, dd, D, lay, causal, phik, V, phiq, dO, dsx, eps);
  a.w = wq;
  a.out = dV;
  a.dx = reinterpret_cast<float*>(w + lay.dphik);
  if ((e = luna::launch_chunk_key(dt, dd, a, s)) != hipSuccess) return hip_fail(e, "key-gradient kernel launch");
  return enqueue_phi_backward(pb, w, lay, Q, K, dQ, dK, grads, s);
}

size_t luna_distill_workspace_bytes(luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                                    const luna_phi_params* p, int32_t param_grads) {
  Problem pb{param_grads ? kOpDistillGrads : kOpDistill, dtype, B, H, n, d, p, 64};
  Layout lay;
  return plan(pb, &lay) == LUNA_OK ? lay.total : 0;
}

luna_status luna_distill(const void* Q, const void* K, luna_dtype dtype, int64_t B, int64_t H, int64_t n, int64_t d,
                         const luna_phi_params* p, int32_t causal, float eps, float* row_loss,
                         const luna_phi_grads* grads, void* ws, size_t ws_bytes, void* stream) {
  g_last_error.clear();
  if (causal != 0 && causal != 1) return fail(LUNA_ERR_INVALID_ARG, "causal must be 0 or 1");
  Problem pb{grads ? kOpDistillGrads : kOpDistill, dtype, B, H, n, d, p, 64};
  Layout lay;
  luna_status st = plan(pb, &lay, ws_bytes);
  if (st != LUNA_OK) return st;
  if (!Q || !K || !row_loss) return fail(LUNA_ERR_INVALID_ARG, "Q, K or row_loss is NULL");
  if (grads && (!grads->W || !grads->b || !grads->fc1_w || !grads->fc1_b || !grads->fc2_w || !grads->fc2_b))
    return fail(LUNA_ERR_INVALID_ARG, "a parameter-gradient array is NULL");
  if (!finite_nonneg(eps)) return fail(LUNA_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if (B * H * ((n + 63) / 64) > ((int64_t)1 << 31) - 1) return fail(LUNA_ERR_UNSUPPORTED, "too many 64-row tiles");
  if ((st = check_ws(lay, ws, ws_bytes)) != LUNA_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  if ((st = enqueue_prepare(pb, w, lay, s)) != LUNA_OK) return st;
  const luna::Dt dt = dtype == LUNA_BF16 ? luna::Dt::BF16 : luna::Dt::F32;
  const int D = p->M * p->L;
  luna::FeatureMapArgs f{};  // features of the queries and keys in the call's dtype, one launch
  f.phi = phi_args(pb, w, lay);
  f.rows_per_head = n;
  f.H = (int)H;
  f.heads = B * H;
  f.X = K;
  f.out = w + lay.phik;
  f.X2 = Q;
  f.out2 = w + lay.phiq;
  hipError_t e = luna::launch_featuremap(dt, dt, (int)d, p->L, f, s);
  if (e != hipSuccess) return hip_fail(e, "feature-map kernel launch");
  luna::DistillArgs a{};
  a.Q = Q;
  a.K = K;
  a.phiq = w + lay.phiq;
  a.phik = w + lay.phik;
  a.stats = reinterpret_cast<float*>(w + lay.dstats);
  a.row_loss = row_loss;
  a.dphiq = grads ? reinterpret_cast<float*>(w + lay.dphiq) : nullptr;
  a.dphik = grads ? reinterpret_cast<float*>(w + lay.dphik) : nullptr;
  a.n = n;
  a.heads = B * H;
  a.causal = causal;
  a.scale = 1.0f / std::sqrt((float)d);
  a.eps = eps;
  a.inv_rows = (float)(1.0 / ((double)B * (double)H * (double)n));
  if ((e = luna::launch_distill(dt, (int)d, D, a, grads != nullptr, s)) != hipSuccess)
    return hip_fail(e, "distillation kernel launch");
  if (!grads) return LUNA_OK;
  return enqueue_phi_backward(pb, w, lay, Q, K, nullptr, nullptr, grads, s);
}

const char* luna_status_string(luna_status s) {
  switch (s) {
    case LUNA_OK: return "ok";
    case LUNA_ERR_INVALID_ARG: return "invalid argument";
    case LUNA_ERR_UNSUPPORTED: return "unsupported problem";
    case LUNA_ERR_WORKSPACE: return "workspace too small";
    case LUNA_ERR_HIP: return "HIP error";
  }
  return "unknown status";
}

const char* luna_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
