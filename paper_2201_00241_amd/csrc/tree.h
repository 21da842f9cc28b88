// The tree path: the triangular solves of many directions as small dense
// products, with the elimination tree cut into nodes (plan: tree.cpp,
// kernels: tree.hip).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "rh_internal.h"

namespace rh {

// Directions of a chunk: the width of a matrix instruction.  A row of a
// chunk's vector is kTreeDirs consecutive values (128 bytes in FP64).
constexpr int kTreeDirs = 16;
// Rows and columns of a tile of a node's matrices.
constexpr int kTreeTile = 16;

// Waves of a leaf and of an upper workgroup.
constexpr int kLeafWaves = 4, kUpperWaves = 16;

// A set of rows of the elimination tree solved by one workgroup: ns rows
// (row0 .. row0 + ns - 1 of the tree order) and nb border rows, the rows above
// the node that its columns reach.  With S its own rows and B the border, a
// node has two matrices of ns + nb rows and ns columns,
//   M = [ T_S^{-1} ; -T_BS T_S^{-1} ],  T = L or U^T (unit diagonal):
// a forward sweep (L, U^T) is M b_S, whose first ns rows are the solution and
// whose others are added to the border rows (the node's update rows), and a
// backward sweep (L^T, U) is M^T [ y_S ; x_B ] with the border rows solved.
// Rows are grouped in tiles of 16, the own rows first (mt tiles), then the
// border rows (bt tiles); columns in mt tiles.  Only tiles that the pattern
// reaches are kept.  An output tile's products (matrix tile times input tile)
// belong to one wave, or above the leaves to successive ones, and a wave's
// products follow each other: wave w takes forward products fwd0 + fwd_at[w]
// .. fwd0 + fwd_at[w + 1] - 1 and the backward products of bwd0 and bwd_at.
// Product p of a list takes matrix tile p, so that a wave reads its matrices
// in one run.  Tile (r, c) of M is forward product map[2 (map0 + r mt + c)] and
// backward product map[... + 1], or -1.
// border0: the border rows' tree positions; u0: its first update row; ent0: its
// rows' ranges of entries (ns + nb + 1 pointers).
struct TreeNode {
  int32_t row0, ns, nb, mt, bt, map0, fwd0, bwd0, border0, u0, ent0;
  uint16_t fwd_at[kUpperWaves + 1], bwd_at[kUpperWaves + 1];
};

// A product of a list: input tile and output tile; whether it is the wave's
// last for the output tile (kProdLast); and, above the leaves, whether the sum
// goes to the wave that holds the output tile's first products (kProdPart), or
// how many of the next waves have parts of it.
constexpr int kProdBits = 8, kProdMore = 2 * kProdBits + 2;
constexpr int32_t kProdMask = (1 << kProdBits) - 1, kProdLast = 1 << (2 * kProdBits), kProdPart = kProdLast << 1;
// Products of a wave: its list is one value per lane, and a leaf's are held in
// registers.
constexpr int kWaveProds = 64, kLeafProds = 6;
// Rows of a leaf node: the products of a node of r rows take about r^2 / 2
// multiplications where substitution takes a few per row, so leaves stay
// small (at 10k buses the tiles of the leaf tier grow from 3,040 at 32 rows
// to 3,833 at 64 and 4,664 at 128); above them every tier is two launches,
// so nodes are as large as one workgroup solves in about the launch's own
// time.
constexpr int kTreeLeafRows = 64, kTreeUpperRows = 256, kTreeTopRows = 448;
// A network of more rows than this has leaves: the fronts of fronts.hip are
// factored by one workgroup each (a tracking step at 200 buses, 379 rows, takes
// 3.06 ms with a single front and 1.64 ms with leaves).
constexpr int kTreeSingleRows = 64;
// Row tiles (own and border) a node may have: a lane group of a workgroup
// stages four own rows and up to eight in all, and a leaf's products fit the
// waves' registers.
constexpr int kLeafTiles = 6, kUpperTiles = 32;

// Offsets within a chunk's memory are 31 bits of bytes.
constexpr int32_t kTreeMaxRows = 1 << 21;

// Update rows of a row's record: at 10k buses none has more than six, at 70k
// few more than eight.
constexpr int kTreeGat = 8;

struct TreePlan {
  bool ok = false;  // false: the network is not taken by this path
  int32_t n = 0, n_u = 0;
  // tiers of nodes, leaves first: nodes tier[t] .. tier[t + 1] - 1; the last
  // tier is one node without border, solved forward and backward at once
  std::vector<int32_t> tier;
  std::vector<TreeNode> nodes;
  std::vector<int32_t> pos;     // factor row -> tree position
  std::vector<int32_t> border;  // tree positions
  // the update rows that the rows above the leaves (from gat0 on, tree order)
  // receive: the first kTreeGat (-1: none), or, where a row receives more,
  // -2 - offset of its list {count, update rows ...} in gat_more as the last
  int32_t gat0 = 0;
  std::vector<int32_t> gat, gat_more;
  // products (see kProdBits), by node and wave
  std::vector<int32_t> fwd, bwd;
  std::vector<int32_t> map;
  // the rows of T_S and T_BS without the diagonal: column (local row), and
  // the positions of the value in the flat factors: lo for L, up / dg (the
  // diagonal) for U^T
  std::vector<int32_t> ent_ptr, lo, up, dg;
  std::vector<uint16_t> col;
  // per column tile of every node {node, column tile}: the work list of the
  // inversion
  std::vector<int32_t> cols;
  std::vector<int32_t> max_tiles;  // per tier: most row tiles (own and border) of a node
  int32_t max_rows = 0;            // most rows (own and border) of a node
};

// Flat factors: row i's L part, then its U part (diagonal first), at
// row_ptr[i].
TreePlan tree_plan(const LuPlan &lu, const std::vector<int32_t> &row_ptr);

}  // namespace rh
