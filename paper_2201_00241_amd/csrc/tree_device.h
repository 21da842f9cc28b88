// Device structures of the tree path, and its host entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "tree.h"

namespace rh {

// A bus of the projection: tangent sources as in the one-workgroup path
// (theta from row tx, -1: reference; v from row vs, or from parameter
// -vs - 1), coefficients, and its incidences.
struct TreeBus {
  int32_t tx, vs, inc0, inc1;
  double ve, sth, sv, pad;
};
struct TreeInc {
  double K, Hps, H, A2, vo;
  int32_t ot, ov;
};

constexpr int kTreeTiers = 12;
// Doubles of a line: chunks start and end at lines.
constexpr int kTreeLine = 32;
// Directions a full Hessian gives one call: the rounds within it keep the
// chip busy, and a call's launches are paid once.
constexpr int32_t kTreeLaunchDirs = 4096;

struct TreeDesc {
  int32_t n_x, n_p, n_bus, n_u, n_slack, n_gp_rows, n_tiers, gat0;
  int32_t tier[kTreeTiers + 1];
  const TreeNode *nodes;
  const int32_t *border, *gat_more, *fwd, *bwd;
  const int4 *gat;
  const double *m64[4];  // the nodes' matrices for the sweeps L, U, U^T, L^T
  const float *m32[4];    // (above the leaves, from product first32 of the lists on)
  int32_t first32[2];     // forward, backward
  const int4 *gp_rows;  // {row, first entry, end, 0} of the rows with entries, ascending
  const int32_t *gp_ptr, *gp_col;  // (all rows' pointers)
  const double *gp_val;
  const int32_t *gpt_ptr, *gpt_row;
  const double *gpt_val, *p_c2x2;
  const TreeBus *bus;
  const TreeInc *inc;
  const int2 *slack_x;  // {tx, vs}
  const double2 *slack_g;
  // G_x and G_x^T by rows, for the residuals of the refined mode
  const int32_t *an_ptr, *an_col, *at_ptr, *at_col;
  const double *an_val, *at_val;
  double norm_n, norm_t;  // their largest row sums
};

// A request's chunks in one round of launches: chunks chunk0 .. chunk0 +
// chunks - 1 of the round.
struct TreeItem {
  const TreeDesc *td;
  const double *W;
  double *HW;
  int64_t ldw, ldhw;
  int32_t k, identity_from, chunk0, chunks, round;
  int32_t at, stride;  // chunk c's place in the scratch is at + c stride, its length stride (in lines of kTreeLine)
  int32_t pad;
  double *rinfo;       // refined mode: 4 doubles per column, or null
};

struct TreeArgs {
  const TreeItem *items;  // n_items of them on the device; null: `one`
  TreeItem one;
  int32_t n_items, n_chunks, norm_iters, lds_rows;
  double tol;
  double *scratch, *norms;
  long long *stamps;
};

struct DevTree;  // a network's plan and device arrays (tree.hip)

// Builds the plan on the first call (false in *used: not for this network),
// and uploads or refreshes the operating point's values.  d_factors: the flat
// factors when they are on the device already, else null.  RH_ENOMEM: there is
// no memory for it, and nothing is kept.
rh_status tree_upload(Network &net, const double *d_factors, bool *used, std::string &err);
// Launches of a forward and a backward sweep: the tiers.
void tree_steps(const DevTree *t, int32_t &fwd, int32_t &bwd);
int64_t tree_bytes(const DevTree *t);

struct TreeRequest {
  DevTree *t;
  const double *W;
  double *HW;
  int64_t ldw, ldhw;
  int32_t k, identity_from;
  double *rinfo;
};
// The requests' chunks in rounds of launches, and the scratch that the
// longest takes: no more than `most` bytes unless one chunk does.  A chunk
// takes what its own network needs, whatever others are in the round.
struct TreeWork {
  std::vector<TreeItem> items;
  int32_t chunks = 0, round = 0, norm_iters = 0;  // round: the most chunks of one
  int64_t data = 0;                               // doubles of a round's chunks; their norms follow
  int64_t norm_doubles() const;                   // of a chunk
  size_t bytes() const;
};
TreeWork tree_work(const std::vector<TreeRequest> &req, int32_t refine, size_t most = SIZE_MAX);
// The launches.  `items`: the work list on the device (null for a single
// request, whose items travel by value).
rh_status tree_launch(const std::vector<TreeRequest> &req, const TreeWork &work, const TreeItem *items, double *scratch,
                      int32_t refine, double tol, long long *stamps, hipStream_t s, std::string &err);

}  // namespace rh
