// Plan of the tree path: the elimination tree of P G_x P^T = L U is cut into
// nodes, in tiers.
//
// Leaf tier: the maximal subtrees of at most kTreeLeafRows rows, several small
// ones sharing a node.  They are independent, and hold nine tenths of the
// rows (at 10k buses).  The rows above are cut the same way into nodes of at
// most kTreeUpperRows rows, and so on until the rest fits one workgroup: the top
// node.  A forward sweep (L or U^T) runs the tiers from the leaves, a backward
// one (U or L^T) from the top; a tier is one launch over all its nodes and
// all directions, and the only ordering across workgroups is that of the
// launches.
//
// Within a node the rows are in postorder, so that a subtree's rows are
// contiguous and the inverse of the node's triangle, whose column j reaches
// j's ancestors only, is zero in most tiles off the subtrees.
#include "tree.h"

#include <algorithm>
#include <stdexcept>

namespace rh {

namespace {

// Border rows up to which small subtrees share a node.
constexpr int32_t kLeafBorder = 32, kUpperBorder = 128;

std::vector<int32_t> postorder(const std::vector<int32_t> &parent) {
  const int32_t n = (int32_t)parent.size();
  std::vector<int32_t> first(n, -1), next(n, -1), post(n), stack;
  for (int32_t v = n - 1; v >= 0; --v)
    if (parent[v] >= 0) {
      next[v] = first[parent[v]];
      first[parent[v]] = v;
    }
  int32_t c = 0;
  for (int32_t r = 0; r < n; ++r) {
    if (parent[r] >= 0) continue;
    stack.push_back(r);
    while (!stack.empty()) {
      const int32_t v = stack.back(), k = first[v];
      if (k >= 0) {
        first[v] = next[k];
        stack.push_back(k);
      } else {
        post[v] = c++;
        stack.pop_back();
      }
    }
  }
  return post;
}

struct Cut {
  std::vector<std::vector<int32_t>> nodes;  // factor rows, in postorder
  std::vector<int32_t> rest;                // ascending
};

// Maximal subtrees of at most R rows of the forest on `rows` (ascending;
// parents above children), neighbours in postorder packed together while
// their rows and borders (a subtree's border is its root's row of U) fit.
Cut cut_forest(const std::vector<int32_t> &rows, const std::vector<int32_t> &parent, const std::vector<int32_t> &post,
               const LuPlan &lu, int32_t R, int32_t border_max) {
  const int32_t n = (int32_t)parent.size();
  std::vector<int32_t> size(n, 0), owner(n, -2), roots;
  for (int32_t v : rows) size[v] = 1;
  for (int32_t v : rows)
    if (parent[v] >= 0) size[parent[v]] += size[v];
  for (size_t q = rows.size(); q-- > 0;) {
    const int32_t v = rows[q], p = parent[v];
    if (size[v] > R) {
      owner[v] = -1;
    } else if (p < 0 || owner[p] == -1) {
      owner[v] = (int32_t)roots.size();
      roots.push_back(v);
    } else {
      owner[v] = owner[p];
    }
  }
  std::vector<int32_t> order(roots.size()), node_of(roots.size());
  for (size_t q = 0; q < roots.size(); ++q) order[q] = (int32_t)q;
  std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return post[roots[a]] < post[roots[b]]; });
  int32_t used = 0, border = 0, nn = 0;
  for (int32_t q : order) {
    const int32_t b = (int32_t)lu.urow[roots[q]].size() - 1;
    if (nn == 0 || used + size[roots[q]] > R || border + b > border_max) {
      ++nn;
      used = border = 0;
    }
    used += size[roots[q]];
    border += b;
    node_of[q] = nn - 1;
  }
  Cut c;
  c.nodes.resize(nn);
  for (int32_t v : rows) {
    if (owner[v] == -1)
      c.rest.push_back(v);
    else
      c.nodes[node_of[owner[v]]].push_back(v);
  }
  for (auto &nd : c.nodes) std::sort(nd.begin(), nd.end(), [&](int32_t a, int32_t b) { return post[a] < post[b]; });
  return c;
}

int32_t tiles_of(int32_t rows) { return (rows + kTreeTile - 1) / kTreeTile; }

}  // namespace

TreePlan tree_plan(const LuPlan &lu, const std::vector<int32_t> &row_ptr) {
  TreePlan plan;
  const int32_t n = plan.n = lu.n;
  if (n <= 0 || n > kTreeMaxRows) return plan;
  const std::vector<int32_t> parent = etree_parent(lu), post = postorder(parent);
  std::vector<int32_t> mark(n, -1);
  int32_t stamp = 0;
  auto border_of = [&](const std::vector<int32_t> &rows) {  // ascending factor rows
    std::vector<int32_t> b;
    ++stamp;
    for (int32_t v : rows) mark[v] = stamp;
    for (int32_t v : rows)
      for (size_t q = 1; q < lu.urow[v].size(); ++q) {
        const int32_t c = lu.urow[v][q];
        if (mark[c] != stamp) {
          mark[c] = stamp;
          b.push_back(c);
        }
      }
    std::sort(b.begin(), b.end());
    return b;
  };
  // tiers
  std::vector<std::vector<std::vector<int32_t>>> tiers;
  std::vector<int32_t> rest(n);
  for (int32_t i = 0; i < n; ++i) rest[i] = i;
  while ((int32_t)rest.size() > (tiers.empty() ? kTreeSingleRows : kTreeTopRows)) {
    const bool leaf = tiers.empty();
    const int32_t most = leaf ? kLeafTiles : kUpperTiles;
    bool done = false;
    for (int32_t R = leaf ? kTreeLeafRows : kTreeUpperRows; R >= 16 && !done; R /= 2) {
      Cut c = cut_forest(rest, parent, post, lu, R, leaf ? kLeafBorder : kUpperBorder);
      bool fits = true;
      for (const auto &nd : c.nodes)
        fits = fits && tiles_of((int32_t)nd.size()) + tiles_of((int32_t)border_of(nd).size()) <= most;
      if (!fits) continue;
      tiers.push_back(std::move(c.nodes));
      rest = std::move(c.rest);
      done = true;
    }
    if (!done && tiers.empty() && n <= kTreeTopRows) break;
    if (!done || tiers.size() > 10) return plan;
  }
  std::sort(rest.begin(), rest.end(), [&](int32_t a, int32_t b) { return post[a] < post[b]; });
  tiers.push_back({rest});  // (possibly without rows)
  // nodes and tree positions
  plan.pos.assign(n, -1);
  plan.tier.push_back(0);
  std::vector<int32_t> local(n, -1), flags;
  std::vector<std::vector<int32_t>> recv(n);
  int32_t row0 = 0;
  for (const auto &T : tiers) {
    int32_t most = 0;
    for (const auto &rows : T) {
      const std::vector<int32_t> bd = border_of(rows);
      TreeNode nd{};
      nd.row0 = row0;
      nd.ns = (int32_t)rows.size();
      nd.nb = (int32_t)bd.size();
      nd.mt = tiles_of(nd.ns);
      nd.bt = tiles_of(nd.nb);
      nd.map0 = (int32_t)plan.map.size() / 2;
      nd.fwd0 = (int32_t)plan.fwd.size();
      nd.bwd0 = (int32_t)plan.bwd.size();
      nd.border0 = (int32_t)plan.border.size();
      nd.u0 = plan.n_u;
      nd.ent0 = (int32_t)plan.ent_ptr.size();
      for (int32_t a = 0; a < nd.ns; ++a) {
        plan.pos[rows[a]] = row0 + a;
        local[rows[a]] = a;
      }
      for (int32_t b = 0; b < nd.nb; ++b) {
        local[bd[b]] = nd.ns + b;
        recv[bd[b]].push_back(nd.u0 + b);
      }
      row0 += nd.ns;
      plan.n_u += nd.nb;
      plan.border.insert(plan.border.end(), bd.begin(), bd.end());  // factor rows for now
      plan.max_rows = std::max(plan.max_rows, nd.ns + nd.nb);
      most = std::max(most, nd.mt + nd.bt);
      // entries of T_S and T_BS by rows: columns j of the node below the row
      auto entries = [&](int32_t i) {
        plan.ent_ptr.push_back((int32_t)plan.col.size());
        for (size_t q = 0; q < lu.lrow[i].size(); ++q) {
          const int32_t j = lu.lrow[i][q];
          if (local[j] < 0 || local[j] >= nd.ns) continue;
          const auto &u = lu.urow[j];
          const int32_t uj = row_ptr[j] + (int32_t)lu.lrow[j].size();
          plan.col.push_back((uint16_t)local[j]);
          plan.lo.push_back(row_ptr[i] + (int32_t)q);
          plan.up.push_back(uj + (int32_t)(std::lower_bound(u.begin(), u.end(), i) - u.begin()));
          plan.dg.push_back(uj);
        }
      };
      for (int32_t v : rows) entries(v);
      for (int32_t v : bd) entries(v);
      plan.ent_ptr.push_back((int32_t)plan.col.size());
      // tiles of M the pattern reaches: column j reaches its ancestors in the
      // node and, through each of them, border rows
      const int32_t nr = nd.mt + nd.bt;
      auto tile_row = [&](int32_t l) { return l < nd.ns ? l / kTreeTile : nd.mt + (l - nd.ns) / kTreeTile; };
      flags.assign((size_t)nr * nd.mt, 0);
      for (int32_t v : rows) {
        const int32_t c = local[v] / kTreeTile;
        for (int32_t a = v; a >= 0 && local[a] >= 0 && local[a] < nd.ns; a = parent[a]) {
          flags[(size_t)tile_row(local[a]) * nd.mt + c] = 1;
          for (size_t q = 1; q < lu.urow[a].size(); ++q) {
            const int32_t l = local[lu.urow[a][q]];
            if (l >= nd.ns) flags[(size_t)tile_row(l) * nd.mt + c] = 1;
          }
        }
      }
      plan.map.resize(plan.map.size() + 2 * (size_t)nr * nd.mt, -1);
      int32_t *map = plan.map.data() + 2 * (size_t)nd.map0;
      const int32_t waves = tiers.size() > 1 && &T == &tiers[0] ? kLeafWaves : kUpperWaves;
      auto assign = [&](int32_t outs, int32_t ins, bool fwd, int32_t first, uint16_t *at, std::vector<int32_t> &list) {
        std::vector<std::vector<int32_t>> of(waves);  // products by wave
        std::vector<int32_t> in;
        auto inputs = [&](int32_t o) {
          in.clear();
          for (int32_t i = 0; i < ins; ++i)
            if (flags[fwd ? (size_t)o * nd.mt + i : (size_t)i * nd.mt + o]) in.push_back(i);
        };
        if (waves == kLeafWaves) {
          // whole output tiles, at most two a wave, longest first to the wave
          // with the fewest products
          std::vector<int32_t> order(outs), cnt(outs), outs_of(waves, 0);
          for (int32_t o = 0; o < outs; ++o) {
            order[o] = o;
            inputs(o);
            cnt[o] = (int32_t)in.size();
          }
          std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return cnt[x] > cnt[y]; });
          for (int32_t o : order) {
            inputs(o);
            if (in.empty()) continue;
            int32_t w = -1;
            for (int32_t q = 0; q < waves; ++q)
              if (outs_of[q] < 2 && (w < 0 || of[q].size() < of[w].size())) w = q;
            ++outs_of[w];
            for (int32_t i : in) of[w].push_back(i | o << kProdBits);
            of[w].back() |= kProdLast;
          }
        } else {
          // equal shares of the products in order of their output tiles: a
          // tile that spans waves is summed up by the first of them
          int32_t all = 0, w = 0;
          for (int32_t o = 0; o < outs; ++o) {
            inputs(o);
            all += (int32_t)in.size();
          }
          const size_t share = std::max(1, (all + waves - 1) / waves);
          for (int32_t o = 0; o < outs; ++o) {
            inputs(o);
            int32_t head = -1;
            for (int32_t i : in) {
              if (of[w].size() == share) {
                if (head >= 0) of[w].back() |= kProdLast | (head < w ? kProdPart : 0);
                ++w;
              }
              if (head < 0) head = w;
              of[w].push_back(i | o << kProdBits);
            }
            if (head < 0) continue;
            of[w].back() |= kProdLast | (head < w ? kProdPart : 0);
            if (head < w) of[head].back() |= (w - head) << kProdMore;
          }
        }
        for (int32_t w = 0; w < waves; ++w) {
          at[w] = (uint16_t)(list.size() - first);
          if (of[w].size() > (size_t)(waves == kLeafWaves ? kLeafProds : kWaveProds)) return false;
          for (int32_t e : of[w]) {
            const int32_t i = e & kProdMask, o = e >> kProdBits & kProdMask;
            map[2 * (fwd ? o * nd.mt + i : i * nd.mt + o) + (fwd ? 0 : 1)] = (int32_t)list.size();
            list.push_back(e);
          }
        }
        at[waves] = (uint16_t)(list.size() - first);
        return true;
      };
      if (!assign(nr, nd.mt, true, nd.fwd0, nd.fwd_at, plan.fwd) ||
          !assign(nd.mt, nr, false, nd.bwd0, nd.bwd_at, plan.bwd))
        return plan;
      for (int32_t c = 0; c < nd.mt; ++c) {
        plan.cols.push_back((int32_t)plan.nodes.size());
        plan.cols.push_back(c);
      }
      for (int32_t v : rows) local[v] = -1;
      for (int32_t v : bd) local[v] = -1;
      plan.nodes.push_back(nd);
    }
    plan.tier.push_back((int32_t)plan.nodes.size());
    plan.max_tiles.push_back(most);
  }
  for (int32_t &b : plan.border) b = plan.pos[b];
  // the updates every row receives, in node order
  plan.gat0 = tiers.size() == 1 ? 0 : plan.tier[1] < (int32_t)plan.nodes.size() ? plan.nodes[plan.tier[1]].row0 : n;
  plan.gat.assign(kTreeGat * ((size_t)n - plan.gat0), -1);
  for (int32_t v = 0; v < n; ++v) {
    const auto &r = recv[v];
    if (r.empty()) continue;
    int32_t *g = &plan.gat[kTreeGat * ((size_t)plan.pos[v] - plan.gat0)];
    const size_t direct = r.size() <= kTreeGat ? r.size() : kTreeGat - 1;
    for (size_t q = 0; q < direct; ++q) g[q] = r[q];
    if (r.size() > kTreeGat) {
      g[kTreeGat - 1] = -2 - (int32_t)plan.gat_more.size();
      plan.gat_more.push_back((int32_t)(r.size() - direct));
      plan.gat_more.insert(plan.gat_more.end(), r.begin() + direct, r.end());
    }
  }
  plan.ok = true;
  return plan;
}

}  // namespace rh
