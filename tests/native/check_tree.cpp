// CPU check of the tree path's plan (compiled and run by tests/test_tree.py).
// Reads a network from a binary file (or, with a number of rows, takes a
// chain, a star or a diagonal of that many rows), forms the nodes' matrices
// from random factors by plain substitution, replays every product list as
// the kernels do (wave by wave, output tiles that span waves summed up by the
// first), and compares the four sweeps with plain row-by-row ones.  Prints
// "max_err <sweep> <value>" and "violations <n>" lines.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2201_00241_amd/csrc/tree.h"

using namespace rh;

template <class T>
static std::vector<T> rd(FILE *f, size_t n) {
  std::vector<T> v(n);
  if (n && fread(v.data(), sizeof(T), n, f) != n) v.clear();
  return v;
}

static int violations = 0;
#define CHECK_THAT(c)                                     \
  do {                                                    \
    if (!(c)) {                                           \
      ++violations;                                       \
      std::printf("violation line %d: %s\n", __LINE__, #c); \
    }                                                     \
  } while (0)

// The matrix of a node (L or U^T) in rows of ns values.
static std::vector<double> node_matrix(const TreePlan &p, const TreeNode &nd, const std::vector<double> &F, bool upper) {
  std::vector<double> m((size_t)(nd.ns + nd.nb) * nd.ns, 0.0);
  for (int a = 0; a < nd.ns + nd.nb; ++a) {
    if (a < nd.ns) m[(size_t)a * nd.ns + a] = 1.0;
    for (int e = p.ent_ptr[nd.ent0 + a]; e < p.ent_ptr[nd.ent0 + a + 1]; ++e) {
      CHECK_THAT(p.col[e] < std::min(a, nd.ns));
      const double v = upper ? F[p.up[e]] / F[p.dg[e]] : F[p.lo[e]];
      for (int j = 0; j < nd.ns; ++j) m[(size_t)a * nd.ns + j] -= v * m[(size_t)p.col[e] * nd.ns + j];
    }
  }
  return m;
}

int main(int argc, char **argv) {
  Context ctx;
  Network net;
  net.ctx = &ctx;
  std::string err;
  LuPlan made;
  const LuPlan *plan = &made;
  if (argc > 2) {
    const int n = std::atoi(argv[2]);
    const std::string kind = argv[1];
    made.n = n;
    made.lrow.resize(n);
    made.urow.resize(n);
    for (int i = 0; i < n; ++i) {
      made.urow[i].push_back(i);
      const int up = kind == "chain" ? i + 1 : kind == "star" ? n - 1 : n;
      if (up > i && up < n) {
        made.urow[i].push_back(up);
        made.lrow[up].push_back(i);
      }
    }
  } else {
    FILE *f = fopen(argv[1], "rb");
    if (!f) return 1;
    const auto hdr = rd<int32_t>(f, 3);
    const int n = hdr[0], m = hdr[1], g = hdr[2];
    const auto bf = rd<int32_t>(f, m), bt = rd<int32_t>(f, m);
    const auto r = rd<double>(f, m), x = rd<double>(f, m), b = rd<double>(f, m);
    const auto ty = rd<int32_t>(f, n);
    const auto pd = rd<double>(f, n), qd = rd<double>(f, n);
    const auto gb = rd<int32_t>(f, g);
    const auto pg = rd<double>(f, g), vg = rd<double>(f, g), c2 = rd<double>(f, g), c1 = rd<double>(f, g),
               c0 = rd<double>(f, g);
    fclose(f);
    const rh_network_desc d{n,         m,         g,         bf.data(), bt.data(), r.data(),
                            x.data(),  b.data(),  ty.data(), pd.data(), qd.data(), gb.data(),
                            pg.data(), vg.data(), c2.data(), c1.data(), c0.data()};
    if (network_build(net, d, err) != RH_OK) return 1;
    plan = &net.lu;
  }
  const LuPlan &lu = *plan;
  const int n = lu.n;
  std::vector<int32_t> rp(n + 1, 0);
  for (int i = 0; i < n; ++i) rp[i + 1] = rp[i] + (int32_t)(lu.lrow[i].size() + lu.urow[i].size());
  const TreePlan p = tree_plan(lu, rp);
  std::printf("ok %d tiers %zu nodes %zu\n", p.ok ? 1 : 0, p.tier.size() - 1, p.nodes.size());
  if (!p.ok) return 0;
  std::mt19937_64 rng(3);
  std::uniform_real_distribution<double> unit(-1, 1);
  std::vector<double> F(rp[n]);
  for (int i = 0; i < n; ++i) {
    const int nl = (int)lu.lrow[i].size();
    for (size_t q = 0; q < (size_t)(rp[i + 1] - rp[i]); ++q) F[rp[i] + q] = 0.2 * unit(rng);
    F[rp[i] + nl] = 1.5 + 0.5 * unit(rng);
  }
  const int tiers = (int)p.tier.size() - 1;
  std::vector<int> owner(n, 0);
  for (int t = 0; t < tiers; ++t)
    for (int id = p.tier[t]; id < p.tier[t + 1]; ++id) {
      const TreeNode &nd = p.nodes[id];
      const bool leaf = t == 0 && tiers > 1, top = t == tiers - 1;
      CHECK_THAT(nd.ns <= (top ? kTreeTopRows : leaf ? kTreeLeafRows : kTreeUpperRows));
      CHECK_THAT(nd.mt + nd.bt <= (top ? kTreeTopRows / kTreeTile : leaf ? kLeafTiles : kUpperTiles));
      CHECK_THAT(nd.mt + nd.bt <= p.max_tiles[t] && nd.ns + nd.nb <= p.max_rows);
      CHECK_THAT(!top || nd.nb == 0);
      CHECK_THAT(t == 0 || nd.row0 >= p.gat0);
      for (int a = 0; a < nd.ns; ++a) ++owner[nd.row0 + a];
    }
  for (int i = 0; i < n; ++i) CHECK_THAT(owner[i] == 1);
  // entry at tile (r, c) of a matrix, rows i, columns j of the tile
  auto local = [](const TreeNode &nd, int r, int i) {
    const int a = r < nd.mt ? r * 16 + i : nd.ns + (r - nd.mt) * 16 + i;
    return a < (r < nd.mt ? nd.ns : nd.ns + nd.nb) ? a : -1;
  };
  const char *names[4] = {"L", "U", "Ut", "Lt"};
  for (int which = 0; which < 4; ++which) {
    const bool fwd = which == 0 || which == 2, upper = which == 1 || which == 2;
    std::vector<double> X(n), ref(n);
    for (int i = 0; i < n; ++i) ref[i] = X[p.pos[i]] = unit(rng);
    if (fwd) {
      for (int i = 0; i < n; ++i)
        for (size_t q = 0; q < lu.lrow[i].size(); ++q) {
          const int j = lu.lrow[i][q];
          const auto &u = lu.urow[j];
          const int k = (int)(std::lower_bound(u.begin(), u.end(), i) - u.begin());
          const int uj = rp[j] + (int)lu.lrow[j].size();
          ref[i] -= (upper ? F[uj + k] / F[uj] : F[rp[i] + q]) * ref[j];
        }
    } else {
      for (int i = n - 1; i >= 0; --i)
        for (size_t q = 1; q < lu.urow[i].size(); ++q) {
          const int j = lu.urow[i][q];
          const auto &l = lu.lrow[j];
          const int k = (int)(std::lower_bound(l.begin(), l.end(), i) - l.begin());
          const int ui = rp[i] + (int)lu.lrow[i].size();
          ref[i] -= (upper ? F[ui + q] / F[ui] : F[rp[j] + k]) * ref[j];
        }
    }
    std::vector<double> upd(p.n_u, 0.0);
    for (int s = 0; s < tiers; ++s) {
      const int t = fwd ? s : tiers - 1 - s;
      const bool leaf = t == 0 && tiers > 1;
      const int waves = leaf ? kLeafWaves : kUpperWaves;
      for (int id = p.tier[t]; id < p.tier[t + 1]; ++id) {
        const TreeNode &nd = p.nodes[id];
        const std::vector<double> m = node_matrix(p, nd, F, upper);
        // what the tiles leave out has to be zero
        for (int r = 0; r < nd.mt + nd.bt; ++r)
          for (int c = 0; c < nd.mt; ++c) {
            if (p.map[2 * (nd.map0 + r * nd.mt + c)] >= 0) continue;
            for (int i = 0; i < 16; ++i)
              for (int j = 0; j < 16 && c * 16 + j < nd.ns; ++j)
                if (local(nd, r, i) >= 0) CHECK_THAT(m[(size_t)local(nd, r, i) * nd.ns + c * 16 + j] == 0.0);
          }
        // input rows by tile row
        const int ins = fwd ? nd.mt : nd.mt + nd.bt, outs = fwd ? nd.mt + nd.bt : nd.mt;
        std::vector<double> in(ins * 16, 0.0), out(outs * 16, 0.0);
        for (int a = 0; a < nd.ns; ++a) {
          in[a] = X[nd.row0 + a];
          if (!fwd || nd.row0 + a < p.gat0) continue;
          const int32_t *g = &p.gat[kTreeGat * (size_t)(nd.row0 + a - p.gat0)];
          for (int q = 0; q < kTreeGat; ++q)
            if (g[q] >= 0) in[a] += upd[g[q]];
          if (g[kTreeGat - 1] <= -2) {
            const int32_t *more = &p.gat_more[-2 - g[kTreeGat - 1]];
            for (int q = 0; q < more[0]; ++q) in[a] += upd[more[1 + q]];
          }
        }
        if (!fwd)
          for (int b = 0; b < nd.nb; ++b) in[nd.mt * 16 + b] = X[p.border[nd.border0 + b]];
        // the waves' lists
        std::vector<std::vector<double>> part(waves);
        std::vector<int> done(outs, 0), head_of(outs, -1), more_of(outs, 0);
        const auto &list = fwd ? p.fwd : p.bwd;
        const uint16_t *at = fwd ? nd.fwd_at : nd.bwd_at;
        std::vector<std::vector<double>> kept(outs);
        for (int w = 0; w < waves; ++w) {
          std::vector<double> acc(16, 0.0);
          int finished = 0;
          CHECK_THAT(at[w + 1] >= at[w] && at[w + 1] - at[w] <= (leaf ? kLeafProds : kWaveProds));
          for (int q = at[w]; q < at[w + 1]; ++q) {
            const int32_t prod = (fwd ? nd.fwd0 : nd.bwd0) + q, e = list[prod];
            const int i = e & kProdMask, o = e >> kProdBits & kProdMask;
            const int r = fwd ? o : i, c = fwd ? i : o;
            CHECK_THAT(i < ins && o < outs);
            CHECK_THAT(p.map[2 * (nd.map0 + r * nd.mt + c) + (fwd ? 0 : 1)] == prod);
            for (int a = 0; a < 16; ++a)
              for (int j = 0; j < 16; ++j) {
                const int la = local(nd, r, a), col = c * 16 + j;
                if (la < 0 || col >= nd.ns) continue;
                const double v = m[(size_t)la * nd.ns + col];
                if (fwd)
                  acc[a] += v * in[c * 16 + j];
                else
                  acc[j] += v * in[r * 16 + a];
              }
            if (!(e & kProdLast)) {
              CHECK_THAT(q + 1 < at[w + 1] && (list[prod + 1] >> kProdBits & kProdMask) == o);
              continue;
            }
            ++finished;
            const int more = e >> kProdMore;
            CHECK_THAT(!leaf || (more == 0 && !(e & kProdPart)));
            if (more) {
              CHECK_THAT(q + 1 == at[w + 1] && head_of[o] < 0);
              head_of[o] = w;
              more_of[o] = more;
              kept[o] = acc;
            } else if (e & kProdPart) {
              CHECK_THAT(part[w].empty() && head_of[o] >= 0 && w <= head_of[o] + more_of[o] && finished == 1);
              part[w] = acc;
            } else {
              CHECK_THAT(!done[o] && head_of[o] < 0);
              done[o] = 1;
              std::copy(acc.begin(), acc.end(), out.begin() + o * 16);
            }
            std::fill(acc.begin(), acc.end(), 0.0);
          }
          CHECK_THAT(!leaf || finished <= 2);
        }
        for (int o = 0; o < outs; ++o) {
          if (head_of[o] < 0) continue;
          for (int w = head_of[o] + 1; w <= head_of[o] + more_of[o]; ++w) {
            CHECK_THAT(w < waves && part[w].size() == 16);
            for (int a = 0; a < 16 && part[w].size() == 16; ++a) kept[o][a] += part[w][a];
          }
          std::copy(kept[o].begin(), kept[o].end(), out.begin() + o * 16);
          done[o] = 1;
        }
        for (int o = 0; o < outs; ++o) CHECK_THAT(done[o]);
        for (int a = 0; a < nd.ns; ++a) X[nd.row0 + a] = out[a];
        if (fwd)
          for (int b = 0; b < nd.nb; ++b) upd[nd.u0 + b] = out[nd.mt * 16 + b];
      }
    }
    double worst = 0.0, scale = 0.0;
    for (int i = 0; i < n; ++i) {
      worst = std::max(worst, std::fabs(X[p.pos[i]] - ref[i]));
      scale = std::max(scale, std::fabs(ref[i]));
    }
    std::printf("max_err %s %.3e\n", names[which], worst / scale);
  }
  std::printf("violations %d\n", violations);
  return 0;
}
