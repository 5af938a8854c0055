// Internal declarations of the level-by-level solver for instances with few
// clusters (multi.hip).
#pragma once

#include "impl.h"

namespace mcc {

// Limits of an instance the kernels take: the clusters fit a mask of eight
// words, one partition's table slice fits the LDS as 32-bit changes, and
// the bitmap of the initial ids fits the LDS of one workgroup.
constexpr int32_t kMultiClusters = 256;
constexpr int32_t kMultiCells = 24576;
constexpr int64_t kMultiVertices = (int64_t)1 << 16;
// Largest instance whose clusters the range kernel counts (its bitmap fits
// the LDS); above kMultiVertices only the count is taken.
constexpr int64_t kMultiCount = (int64_t)1 << 20;

// Counters and verdicts of one instance.
struct MultiCtl {
  int32_t K0;         // consensus clusters
  int32_t lmax;       // largest label value
  int32_t err;        // kErr* bits
  int32_t done;
  int32_t nprop;      // proposals of the current pass
  int32_t passes, converged, fallback_rounds, clusters;
  int32_t stage;      // 1: the batch did not lower the objective; the second
                      // slot of the pass commits its conflict-free subset
  int64_t pass_evals, pass_boundary;
  int64_t evals, boundary, moves;
  int64_t O, O0;      // objective, and the initial one
  int64_t dN2, dS2;   // changes of the sums of squares by the current pass
};

// One instance (device copy).  The table holds one slice per partition,
// slice i at N + i * cs: a row of rs counts per label value, N_i(x, l) at
// l * rs + x, in int16 when the instance has fewer than 2^15 vertices, else
// int32.  Rows are an odd number of 16-byte units, so that consecutive rows
// start in different LDS banks.  A multiple of 16 bytes, as an upload of one
// instance then is too: copies of other sizes took 0.4 us longer.
struct alignas(16) MultiInst {
  int64_t n;
  const int64_t* row_ptr;
  const int32_t* col;
  const int32_t* const* labels;  // k device pointers
  const int32_t* init;           // null: singletons
  int32_t* out;
  uint16_t* C;
  int32_t* rawid;
  int2* plist;       // proposals of the pass: (vertex, target)
  int64_t* dprop;    // their gains
  int32_t* s;
  void* N;
  int32_t k;
  int32_t K0, Ls;
  int32_t rs, cs;    // entries between two rows, between two slices
  int32_t pad;
};

struct MultiItem {
  int32_t inst, part;  // instance, and the tile or partition of it
};

struct MultiArgs {
  const MultiInst* inst;
  MultiCtl* ctl;
  int32_t count;        // instances
  int32_t max_rounds;
  int32_t literal;
  int32_t pad;
  int64_t* trace;       // device int64[4 * max_rounds] of a lone instance, or null
};

// Comparison of the clusters of a lone instance with its one partition, from
// its table (the statistics mcc_compare reports, and the distinct labels).
struct MultiCompare {
  int64_t rowmax, colmax;  // sums of the rows' and the columns' largest counts
  double cells, rows, cols;  // sums of c ln c over the cells, clusters, labels
  int32_t labels;            // labels that occur
  int32_t pad;
};
void launch_multi_compare(const MultiArgs& a, int32_t Ls, MultiCompare* out, hipStream_t st);

// First-occurrence relabelling of up to kMultiCanon ids in [0, n) by one
// workgroup; *total: the distinct ids, or -1 if one lies outside [0, n) (then
// nothing is written).
constexpr int64_t kMultiCanon = 16384;
void launch_multi_canonical(const int32_t* in, int64_t n, int32_t* out, int32_t* total,
                            hipStream_t st);

// Dynamic LDS of the scorer: offsets, clusters, masks of `words` words a
// vertex, cluster sizes, and the slice buffer.
size_t multi_score_lds(int tile, int words, size_t slice_bytes);

// Clusters of every instance (C, rawid, K0) and the label ranges: workgroups
// [0, count) take an instance's clusters, the others one (instance,
// partition) of `labels` each.
// n_max: the largest instance.
void launch_multi_ranges(const MultiArgs& a, const MultiItem* labels, int32_t nlabels,
                         int64_t n_max, hipStream_t st);
void launch_multi_build(const MultiArgs& a, const MultiItem* parts, int32_t nparts, bool wide,
                        int32_t cells_max, hipStream_t st);
// mode: how the instances of the list are scored (multi_score_mode, below
// kMultiModes).
constexpr int kMultiModes = 4, kMultiDirect = 1;
int multi_score_mode(int32_t K0, int32_t cs, bool wide, int tile);
void launch_multi_score(const MultiArgs& a, const MultiItem* tiles, int32_t ntiles, bool wide,
                        int mode, int tile, int words, size_t slice_bytes, hipStream_t st);
void launch_multi_apply(const MultiArgs& a, const MultiItem* parts, int32_t nparts, bool wide,
                        int32_t cells_max, hipStream_t st);
void launch_multi_commit(const MultiArgs& a, const int32_t* ids, int32_t nids, hipStream_t st);

}  // namespace mcc
