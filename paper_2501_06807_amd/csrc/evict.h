// Launch interface of the static-eviction kernels.
#pragma once
#include "common.h"

namespace mpc {

constexpr int kNumXcd = 8;       // accelerator dies; workgroup i runs on die i % 8
constexpr int kRowBlock = 256;      // window rows per row-statistics workgroup
constexpr int kColBlockKeys = 256;  // keys per column-sum workgroup (its waves share each staged row tile)
constexpr int kColThreads16 = 256;  // column-sum workgroup for 16-bit inputs: 4 waves of 64 keys
constexpr int kRowThreads16 = 256;  // row-statistics workgroup for 16-bit inputs: 4 waves of 64 rows

struct EvictArgs {
  const void* q_win;   // [L][B][Hq][W][d]
  const void* k;       // [L][B][Hkv][T][d]
  const void* v;
  int32_t* kept;       // [L][B][Hkv][keep]
  void* k_out;         // [L][B][Hkv][out_rows][d], rows [0, keep) written
  void* v_out;
  float* score;        // [L][B][Hkv][T] accumulated attention (token_score or workspace)
  float2* rowstat;     // [L][B][Hq][W]: (whole-number offset b, every fma(c, score, b) <= 1; 1 / sum of exp2(fma(c, score, b)))
  float* row_lse;      // [L][B][Hq][W] natural log-sum-exp, optional
  double2* part;       // row pass partials [owner heads][splits][W]: (sum, offset); unused with one split
  int splits;          // workgroups that share a row block's keys
  double* col_part;    // column pass partials [owner heads][col_splits][T]; unused with one split
  int col_splits;      // workgroups that share a key block's window rows
  int col_group;       // 16-bit column-pass units whose key blocks are dealt together (col_group below)
  int B, layer0, n_layers, Hq, Hkv, T, W, keep, local_keep, causal, period, start;
  int out_rows;        // row capacity of k_out / v_out per (layer, sequence, kv head)
  OwnerTable own;      // owner layers of the block
  uint64_t skip[kMaxLayers / 64];  // layers whose rows the gather leaves to the cluster build (bit l)
  float c32;           // fp32(sm_scale * log2(e)), the exponent scale of both scoring passes
};

constexpr int kMaxRowSplits = 16;
constexpr int kSplitTiles = 2;  // what a split costs beside its tiles, in tiles

// Workgroups per row block of the row pass for `heads` owner query heads.
int row_splits(int heads, int T, int W, int causal);

constexpr int kMaxColSplits = 16;

// Workgroups per key block of the column pass for `heads` owner kv heads of `group` query heads.
int col_splits(int heads, int T, int W, int group);

// Units (owner kv heads times row splits) of the 16-bit column pass to a group; unit_bytes: window rows a unit reads.
int col_group(int units, int T, int64_t unit_bytes);

hipError_t launch_rowstats(const EvictArgs& a, int dtype, int D, hipStream_t st);
hipError_t launch_colsum(const EvictArgs& a, int dtype, int D, hipStream_t st);
hipError_t launch_topk(const EvictArgs& a, hipStream_t st);
hipError_t launch_gather(const EvictArgs& a, int dtype, int D, hipStream_t st);

}  // namespace mpc
