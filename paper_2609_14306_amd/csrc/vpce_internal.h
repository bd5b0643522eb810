// Internal interface between the host API (vpce_api.cpp) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "vpce.h"

namespace vpce {

// Vocabulary shards in visiting order: position i is shard order[i].
struct ShardTable {
  const void* w[VP_MAX_SHARDS];   // device [rows[i], d]
  int64_t off[VP_MAX_SHARDS];     // global id of the shard's first row
  int32_t rows[VP_MAX_SHARDS];    // V_p
  int32_t tile0[VP_MAX_SHARDS + 1];  // first forward tile index of position i (prefix sums)
  int32_t P;
};

struct FwdArgs {
  ShardTable st;
  const void* H;
  const int64_t* targets;
  int64_t T;
  int32_t d;
  int32_t n_tok_blocks, n_splits, n_tiles;
  int32_t kind;                 // tile of the kernel (see fwd_tile)
  unsigned long long* counter;  // cleared by the kernel for the merge that follows; may be null
  float* m_part;  // [n_splits][T]
  float* s_part;  // [n_splits][T]
  float* y_tgt;   // [T]
};

struct CombArgs {
  const float* m_part;
  const float* s_part;
  const float* y_tgt;
  const int64_t* targets;
  int64_t T, V, ignore_index;
  int32_t n_splits;
  float* loss;
  float* lse;
  unsigned long long* bad_counter;
};

// Per-token fold state of Algorithm 2 as the ABI exposes it: float32 [3][T],
// planes m (running maximum logit, natural units), s (sum of e^(y - m) over the
// ids folded so far) and y (the target logit once its shard has been folded).
struct FoldArgs {
  const float* m_part;  // [n_splits][T], base-2 domain (max of y log2 e)
  const float* s_part;  // [n_splits][T]
  int64_t T;
  int32_t n_splits;
  float* state;
};

struct FinArgs {
  const float* state;
  const int64_t* targets;
  int64_t T, V, ignore_index;
  float* loss;
  float* lse;
  unsigned long long* bad_counter;
};

struct GradArgs {
  const void* W;   // first row of this vocabulary chunk, [M, d]
  const void* H;   // whole H [T, d]
  const int64_t* targets;
  const float* lse;
  const float* grad;
  // The residual strip in two layouts, Tc tokens by Vc vocabulary rows each,
  // k-blocked in 128-byte blocks of KB elements (64 bfloat16, 32 float32):
  // G [Tc/KB][Vc][KB] (element (v, t) at ((t / KB) Vc + v) KB + t % KB) and
  // G^T [Vc/KB][Tc][KB] (element (t, v) at ((v / KB) Tc + t) KB + v % KB), so that a
  // KB-deep slice of a 256-row tile of either operand is one contiguous 32 KiB block.
  void* strip;
  void* strip_t;
  int64_t Tc, Vc;
  int64_t t0;      // first token of this chunk
  int64_t gid0;    // global id of the chunk's first row
  int64_t V, ignore_index;
  const float* yt;  // [T] target logit h_t . w_{targets[t]} of every token (0 if none)
  int32_t M;       // vocabulary rows in this chunk
  int32_t N;       // tokens in this chunk
  int32_t d;
  int32_t n_vt;    // vocabulary tiles over M
};

// Target logits: yt[t] = h_t . w_{targets[t]} for targets in [0, V), 0 otherwise.  The
// shard table may list the shards in any order.
struct TgtArgs {
  ShardTable st;
  const void* H;
  const int64_t* targets;
  int64_t T, V;
  int32_t d;
  float* yt;
  // when not null: set to the number of targets outside [0, V) that are not ignore_index
  // (counted by one workgroup: for few tokens)
  unsigned long long* count;
  int64_t ignore_index;
};

// out[c][r] = in[r][c] for r < R (zero for R <= r < R_pad), c < C.  in is
// row-major with pitch ld_in; out is k-blocked in 128-byte blocks of KB elements
// (64 bfloat16, 32 float32), [R_pad/KB][C][KB] (element (c, r) at
// ((r / KB) C + c) KB + r % KB).  C and ld_in are whole 16-byte vectors, R_pad a
// multiple of KB.
struct TransposeArgs {
  const void* in;
  int64_t ld_in;
  void* out;
  int32_t R, C, R_pad;
};

struct TileShape {
  int bm, bn;  // the large tile: vocabulary rows by tokens
  int kblock;  // elements of one 128-byte k-block of the backward workspaces
};

TileShape tile_shape(int dtype);

// One launch of the backward (bwd_stage_kernel): the residual tiles of strip k and the dH
// and dW tiles of strip k - 1.  A strip is one token chunk of whole shards, or of one
// balanced piece of a large shard: its segments, in visiting order, each starting at a
// strip row that is a multiple of the residual tile's rows.  The dH tiles of a strip
// run over all its segments, or are split into jobs along the vocabulary (where there
// are few of them and their sums are long), each with a partial dH of its own.
constexpr int kMaxSegs = 16, kMaxJobs = 32;
struct StageSeg {
  const void* w;   // its first row, [rows, d]
  float* dw;
  int64_t gid0;        // global id of the first row
  int32_t rows, row0;  // rows, and the strip row that the first of them has
};
// n_seg segments from `seg` on; one alone may be a part: rows k0 .. k0 + rows - 1 of it
// (k0 in whole k-blocks).
struct StageJob {
  int32_t seg, n_seg, k0, rows, beta;
};
struct StageArgs {
  GradArgs g;  // residual tiles (W, gid0, M are the segments'); d, Tc, Vc of both strips
  StageSeg gseg[kMaxSegs], cseg[kMaxSegs];  // of the strip written and of the one contracted
  StageJob job[kMaxJobs];
  int32_t n_gseg, n_cseg, n_job;
  int32_t w_tiles;   // dW row tiles of the strip contracted
  int32_t order[3];  // kinds (0 dH, 1 dW, 2 residual) in launch order
  int32_t beta_w;    // dW is added to
  int64_t c_t0;      // token chunk of the strip contracted
  int32_t c_N;
  const void *G, *Gt;  // its residual
  const void *Wt, *Ht;  // class 3: k-blocked transposed copies of its W rows and of H
  float* part;         // [jobs][T][d], or dH itself for one job
  int64_t part_stride;
};
// Tile classes: 0 (bfloat16): 256 x 256 tiles; 1: 128 x 64 ones; 2: 128 x 128 ones, all of
// them with W and H read transposed; 3: 256 x 256 tiles on transposed copies.
struct BwdTile {
  int bm, bn;    // residual tile: vocabulary rows by tokens; the contractions' tiles are
                 // bm columns of d by bn rows
  double us;     // time per 128-byte slice of a tile with every CU at work
};
BwdTile bwd_tile(int dtype, int cls);
int bwd_col_blocks(int cls, int d);  // column blocks of the contractions
bool run_stage(int dtype, int cls, const StageArgs& a, hipStream_t s);
// out[i] = sum over k < n of part[k * len + i], in the order of k; len % 4 == 0
bool run_sum_parts(const float* part, int n, int64_t len, float* out, hipStream_t s);

// Tiles the forward can run on: kind 0 is the 256 x 256 tile of every large problem,
// the others are the streamed tiles for few tokens.
constexpr int kFwdKinds = 3;
struct FwdTile {
  int bm, bn;             // vocabulary rows by tokens
  int per_cu;             // workgroups a CU holds
  double shared, stream;  // time per slice: W shared by several token blocks, or by none
};
FwdTile fwd_tile(int dtype, int kind);

// Bytes of the library-owned device workspace of vp_ce_forward_noalloc.
constexpr size_t kScratchBytes = 16u << 20;
// Device address of that workspace on the current device (looked up on the first
// call per device and kept); false if the lookup fails.
bool scratch_base(void** out);
bool run_ws_init(unsigned long long* counter, hipStream_t s);
bool run_fill_zero(float* p, int64_t n, hipStream_t s);
bool run_fwd(int dtype, const FwdArgs& a, hipStream_t s);
bool run_comb(const CombArgs& a, hipStream_t s);
bool run_state_init(float* state, int64_t T, hipStream_t s);
bool run_fold_merge(const FoldArgs& a, hipStream_t s);
bool run_fold_finalize(const FinArgs& a, hipStream_t s);
bool run_count_bad(const int64_t* targets, int64_t T, int64_t V, int64_t ignore_index,
                   unsigned long long* counter, hipStream_t s);
// Per-XCD tile counts of one backward stage launch (dH, dW, residual tiles).
struct StageSplit {
  int32_t cnt[3][8], first[3][8];
};

bool run_transpose(int dtype, const TransposeArgs& a, hipStream_t s);
bool run_target_logits(int dtype, const TgtArgs& a, hipStream_t s);

}  // namespace vpce
