// Declarations of the kernels around the scans (dresd_merge.hip,
// dresd_transform.hip, dresd_drafts.hip, dresd_parts.hip, dresd_kmeans.hip),
// shared with the host runtime.  The scan kernels do not include this file.
#pragma once
#include "dresd_internal.h"

namespace dresd {

struct MergeParams {
  const uint64_t *lists;     // [B][G][C] from the scan
  const uint32_t *lcnt;      // [B][G]
  const uint64_t *lkth;      // [B][G]
  const uint64_t *lfirst;    // [B][G]
  uint64_t *spill;           // [B][spill_cap] candidates past the LDS cache
  int64_t spill_cap;
  int B, k, C, G;
  uint64_t *tau_out;         // sample mode: k-th best key per query, else tau_fb (0 if none)
  const uint64_t *tau_fb;    // sample mode: the bound the pass's sample falls back to (may be null)
  uint64_t *spec_out;        // sample mode: spec_rank-th best key per query (may be null)
  int spec_rank;             // 1 <= spec_rank <= k when spec_out is set
  int64_t *idx;              // final mode outputs
  float *score;
  int32_t *tokens;           // may be null
  const int32_t *cont;       // [N, L]
  int64_t N;                 // rows of cont: a winner outside [0, N) is written as (-1, -inf, 0)
  int L;
  int final_mode;
};

// Query-side transform (dresd_transform.hip): y = unit rows of
// ((x - mean) / sqrt(var + eps_z)) W.
struct TransformParams {
  const float *x;            // [M, D]
  const float *mean, *var;   // [D]
  const float *W;            // [D, l] row-major
  float *y;                  // [M, l]
  float *part;               // [splits][M][l] partial sums (splits > 1)
  int64_t M;
  int D, l;
  int splits, dslice;        // D split into `splits` slices of `dslice` dims
  float eps_z, eps_n;
};
// Splits of D for an M x l output on a device with `cus` compute units.
int transform_splits(int64_t M, int D, int l, int cus);
hipError_t launch_transform(const TransformParams &p, hipStream_t st);
// Its second kernel alone: adds the partial sums (splits > 1), unit rows.
hipError_t launch_finish_rows(const TransformParams &p, hipStream_t st);

// Datastore-sized batches on the 16-bit matrix cores (dresd_project.hip).
struct ProjectParams {
  TransformParams t;         // splits: slices of whole 32-dim blocks (dslice unused)
  void *op;                  // weight operands
  float *norm;               // [KB][64] means and factors of a block's dims
  float *wmax;               // per workgroup of the operand kernel: the largest weight
  int KB, NT, groups;        // 32-dim blocks, column tiles per workgroup, column groups
  int64_t off_norm, off_wmax, off_part, bytes;  // workspace
};
// Whether a batch runs there, and its shape and workspace.
bool project_split_plan(int64_t M, int D, int l, int cus, ProjectParams *out);
hipError_t launch_project_split(ProjectParams &p, void *ws, hipStream_t st);

// Draft assembly (dresd_drafts.hip): tokens [B, k, L] -> drafts [B, r, length],
// count [B].
struct DraftParams {
  const int32_t *tokens;
  int32_t *drafts, *count;
  int B, k, L, r, length, eos;
};
hipError_t launch_pack_drafts(const DraftParams &p, hipStream_t st);

// Probed segments of a partitioned search (dresd_parts.hip): one workgroup
// per query turns its probe list into seg_off / seg_tile.
struct SegParams {
  const int64_t *probes64;   // [B][S] partition ids (one of the three is set)
  const int32_t *probes32;
  const int32_t *tok;        // [P] ascending first tokens, partition p holding tok[p]; with
  const int32_t *next_tok;   //   next_tok [B] each query probes its token's partition (S = 1)
  const int32_t *part_tile;  // [P + 1] first tile of each partition
  int32_t *seg_off, *seg_tile;
  int B, S, P;
};
hipError_t launch_segments(const SegParams &p, hipStream_t st);
// Tiled layout of the keys and first-token column (dresd_layout.hip).
struct LayoutParams {
  const void *src;           // [N, d] row-major
  void *dst;                 // tiles
  const uint32_t *slot_row;  // partitioned layout: row of each slot (null: slot = row)
  int64_t N, tiles;
  int d, KB;
};
hipError_t launch_layout(const LayoutParams &p, int dtype, int cus, hipStream_t st);
hipError_t launch_first_tokens(const int32_t *cont, int L, int64_t n, int64_t nslot, int32_t *out,
                               hipStream_t st);
// Grouping of rows into partitions (dresd_group.hip).
constexpr int kGroupTile = 4096;  // rows per workgroup of a sort pass
struct GroupParams {
  const int32_t *cont;       // by token: [n, L] values, the key is the first token; else null
  const int32_t *assign;     // else [n] partition of each row
  const int32_t *values;     // [n, L] values (first tokens of the slots)
  int64_t n, nblk, nslot;    // rows, blocks of kGroupTile rows, slots
  int L, P, by_token;
  // temporary memory: the keys and rows before and after a pass (`src` holds
  // the current ones), digit histograms [4][256], positions [256][nblk]
  uint32_t *key[2], *row[2];
  uint32_t *hist, *counts;
  uint32_t *bad, *distinct;  // an assignment outside [0, P); number of distinct keys
  int src, shift, first;
  uint32_t *start;           // [P + 1] first sorted position of each partition
  int32_t *tok;              // by token: [P] the partitions' tokens
  const int32_t *part_tile;  // [P + 1] first tile of each partition
  uint32_t *slot_row;        // [nslot] out
  int32_t *ftok_slot;        // [nslot] out
};
hipError_t launch_group_keys(GroupParams &p, hipStream_t st);
hipError_t launch_group_pass(GroupParams &p, int digit, bool first, hipStream_t st);
hipError_t launch_group_distinct(GroupParams &p, hipStream_t st);
hipError_t launch_group_bounds(GroupParams &p, hipStream_t st);
hipError_t launch_group_slots(GroupParams &p, hipStream_t st);
hipError_t launch_iota(int32_t *out, int64_t n, hipStream_t st);
// Spherical k-means (dresd_kmeans.hip).
struct KmeansParams {
  const void *x;             // [n, d] rows, storage type dtype
  int64_t n;
  int d, dtype, P;
  const float *centroids;    // [P, d] (assign)
  int32_t *assign;           // [n] out (assign)
  float *score;              // [n] out, may be null (assign)
  const int32_t *assign_in;  // [n] (update)
  float *centroids_out;      // [P, d] in/out (update)
  int32_t *counts;           // [P] out, may be null (update)
  long long *sums;           // [P, d] fixed-point workspace (update)
  int32_t *cnt;              // [P] workspace (update)
  const uint32_t *sorted_row, *sorted_part;  // rows in partition order (update, may be null)
  int64_t offset;            // first picked row, in [0, n) (init)
  // assign only the rows marked -1, listed from this many rows at a time, after
  // unpacking (score, id) keys [n] (may be null)
  int chunk;
  const uint64_t *packed;
};
// Assignment on the 16-bit matrix cores (dresd_assign.hip).
struct AssignParams {
  const void *x;             // [n, d] rows, storage type dtype
  const float *centroids;    // [P, d]
  int32_t *assign;           // [n] out; -1: the row is left to the fp32 path
  float *score;              // [n] out, may be null
  int64_t n;
  int d, dtype, P;
  int KB;                    // blocks of 32 dims, rounded up to a built variant
  int ppad;                  // P rounded up to whole groups of 64
  int splits;                // workgroups that share a block of rows
  // workspace: centroid operands, each centroid's score factor, per centroid
  // tile whether it needs the fp32 path, and (splits > 1) [n] packed results
  void *op;
  float *scale;
  int32_t *special;
  uint64_t *packed;
  int64_t off_scale, off_special, off_packed, bytes;
};
constexpr int64_t kAssignMaxOperand = (int64_t)256 << 20;  // bytes of centroid operands
// Whether rows of this width run there, and the call's shape and workspace.
bool assign_split_plan(int64_t n, int d, int dtype, int P, int cus, AssignParams *out);
hipError_t launch_assign_split(AssignParams &p, void *ws, hipStream_t st);
// The fp32 assignment; with `left` only the rows it marks with id -1 (taking
// the ids and scores of the others from left->packed first, if set).
hipError_t launch_kmeans_assign(const KmeansParams &p, const AssignParams *left, int cus,
                                hipStream_t st);
hipError_t launch_kmeans_update(const KmeansParams &p, int cus, hipStream_t st);
hipError_t launch_kmeans_init(const KmeansParams &p, hipStream_t st);

}  // namespace dresd
