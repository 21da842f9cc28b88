// P G_x P^T = L U by dense fronts (multifrontal, static diagonal pivots).
//
// Row by row, the factorisation is a chain of elimination steps as long as
// the rows at the top of the tree are wide: 3.1 ms of 3.5 at 10k buses, in one
// workgroup.  Here every node of the tree plan (tree.h) has a front, the
// dense matrix of its own rows S and its border B; the entries of G_x and
// what is left of the fronts below are summed into it, the rows of S are
// eliminated, and the rest (B, B) waits for the nodes above.  A tier is two
// launches, so that the chain is a few dozen panels of 16 columns.
//
// Fronts are stored in tiles of 16 x 16 (own rows first, then the border, as
// in the plan), row-major in a tile.  A panel's diagonal tile is factored by
// one wave in registers, its rows of L and columns of U by substitution, one
// per thread, and the rest of the front takes the panel's product on the
// matrix cores.  The mismatch g is one more column of the front, so that L y =
// P g comes with the factorisation, and the Newton step is the sweep with U
// from the top down, a launch per tier.
//
// Measured before and after: the factorisation 3.5 ms and 0.43 ms at 10k buses
// (leaves 31 us, the tier above 240, the top 125), 0.60 ms and 0.13 ms at 1k; the
// two triangular solves by levels 0.46 ms and 0.05 ms at 10k (top 21 us, the
// tier below 23, leaves 9), 0.16 ms and 0.02 ms at 1k.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <limits>
#include <memory>

#include "fronts.h"
#include "tree.h"

namespace rh {

namespace {

#define HIP_TRY(expr)                                                          \
  do {                                                                         \
    hipError_t e_ = (expr);                                                    \
    if (e_ != hipSuccess) {                                                    \
      err = std::string(#expr) + ": " + hipGetErrorString(e_);                 \
      return RH_EDEVICE;                                                       \
    }                                                                          \
  } while (0)

constexpr int kT = kTreeTile, kTT = kT * kT;
typedef double v4d __attribute__((ext_vector_type(4)));

struct FrontNode {
  int64_t f0;            // first value of the front
  int32_t ns, nb, mt, nt;  // own and border rows; tiles of own rows, and of all
  int32_t a0, a1;        // leaves: entries of G_x
  int32_t row0, border0;  // tree position of the own rows, place in the list of the border's
};

// Lane C of each group of 16 lanes to all its lanes.
template <int C>
__device__ __forceinline__ double group_bcast(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + C, 0xF, 0xF, true);
}
// Columns C .. 0 of the back substitution with a 16 x 16 triangle: lane r of
// each group holds v_r and row r right of the diagonal, rl = 1 / U(r, r).
template <int C>
__device__ __forceinline__ void back_steps(double &v, const double (&d)[kT], double rl) {
  v = fma(-d[C], group_bcast<C>(v * rl), v);
  if constexpr (C > 0) back_steps<C - 1>(v, d, rl);
}

// Columns C .. 14 of the substitution with a unit lower triangle: lane r holds
// v_r and row r left of the diagonal.
template <int C>
__device__ __forceinline__ void forward_steps(double &v, const double (&l)[kT]) {
  if constexpr (C + 1 < kT) {
    v = fma(-l[C], group_bcast<C>(v), v);
    forward_steps<C + 1>(v, l);
  }
}

// Sum over the 16 lanes of each group, in all of them.
template <int R>
__device__ __forceinline__ double rotate(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + R, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + R, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double group_sum(double v) {
  v += rotate<8>(v);
  v += rotate<4>(v);
  v += rotate<2>(v);
  return v + rotate<1>(v);
}

// 1 / d for a pivot d: the hardware reciprocal (to 2^-23) and two Newton
// steps, the last of which leaves the rounding of one operation; a division's
// scaling and fix-up, for denormal and infinite pivots (which the pivot test
// refuses), would double the chain.
__device__ __forceinline__ double pivot_rcp(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}

// Step C of L U of a 16 x 16 tile: lane c of each group of 16 lanes holds
// column c, register r its entry r (L not yet divided by the pivots; rl: the
// reciprocal of the lane's own).  The groups do the same, so that every
// broadcast stays within one.  The empty asm statements materialise d[r] at
// the end of the step: the compiler would otherwise sink each entry's updates
// down to its own step, where they are a serial chain.
template <int C>
__device__ __forceinline__ void tile_lu(double (&d)[kT], double &rl, int l16) {
  if constexpr (C < kT) {
    const double rp = pivot_rcp(group_bcast<C>(d[C])), u = l16 > C ? d[C] : 0.0;
    rl = l16 == C ? rp : rl;
#pragma unroll
    for (int r = C + 1; r < kT; ++r) d[r] = fma(-(group_bcast<C>(d[r]) * rp), u, d[r]);
#pragma unroll
    for (int r = C + 1; r < kT; ++r) asm volatile("" : "+v"(d[r]));
    tile_lu<C + 1>(d, rl, l16);
  }
}

// The next panel's diagonal tile (in a wave's registers as the matrix
// instructions leave it) factored, to LDS and back to the front.  Rows past
// the node's own (`own` of the tile are) get a unit diagonal.
__device__ __forceinline__ void front_diag(v4d t, double *T, double *D, double *dinv, int32_t own, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) D[r * 64 + lane] = 4 * r + g < own ? t[r] : 4 * r + g == l16 ? 1.0 : 0.0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  double d[kT], rl = 0.0;
#pragma unroll
  for (int r = 0; r < kT; ++r) d[r] = D[r * kT + l16];
  tile_lu<0>(d, rl, l16);
  // a quarter of the rows from each group
  if (g == 0) dinv[l16] = rl;
#pragma unroll
  for (int r = 0; r < kT; ++r) {
    if ((r & 3) != g) continue;
    const double v = r > l16 ? d[r] * rl : d[r];
    D[r * kT + l16] = v;
    T[r * kT + l16] = v;
  }
}

// A node's own rows eliminated, 16 columns (a panel) at a time.  NW waves: a
// panel has at most 2 * 16 * (nt - 1) rows of L and columns of U, one per
// thread.  LDS: the panel (a row's 16 values of L in steps of 16, a column's
// of U likewise, as the matrix instructions read them) and the diagonal
// tiles.  The first wave factors the next diagonal tile while the others
// take the product.  LEAF: the front is cleared and G_x's entries are put in
// first (no front below).  What bounds it: a panel is a chain of a trip to
// L2, a substitution of 16, and of 16 pivots or the product, whichever is
// longer: one CU's matrix cores and path to L2 in the large fronts.
//
// The right-hand side, after the front's tiles: in LDS meanwhile; own rows end
// as y, the border's as what is left for the fronts above.
template <int NW, bool LEAF>
__global__ __launch_bounds__(NW * 64) void front_factor(double *fronts, const FrontNode *nodes, int32_t node0,
                                                        const int32_t *a_dst, const int32_t *a_src,
                                                        const int32_t *row_g, const double *gx, const double *grhs) {
  extern __shared__ __align__(16) double lds[];
  const FrontNode nd = nodes[node0 + blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double *F = fronts + nd.f0;
  const int nt = nd.nt, mt = nd.mt;
  double *Dall = lds, *Y = Dall + 2 * (kTT + kT), *R = Y + kT, *Lp = R + nt * kT, *Up = Lp + (nt - 1) * kTT;
  double *Rf = F + (int64_t)nt * nt * kTT;
  for (int r = tid; r < nt * kT; r += NW * 64) {
    if constexpr (LEAF)
      R[r] = r < nd.ns ? grhs[row_g[nd.row0 + r]] : 0.0;
    else
      R[r] = r < nd.ns ? Rf[r] : 0.0;
  }
  auto tile_at = [&](int i, int j) { return F + (int64_t)(i * nt + j) * kTT; };
  if constexpr (LEAF) {
    for (int i = tid; i < nt * nt * kTT; i += NW * 64) F[i] = 0.0;
    __syncthreads();
    for (int32_t e = nd.a0 + tid; e < nd.a1; e += NW * 64) F[a_dst[e]] = gx[a_src[e]];
    __syncthreads();
  }
  if (wave == 0 && mt > 0) {
    v4d t;
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = F[r * 64 + lane];
    front_diag(t, F, Dall, Dall + kTT, nd.ns, lane);
  }
  __syncthreads();
  for (int k = 0; k < mt; ++k) {
    const int n1 = nt - k - 1;
    const double *D = Dall + (k & 1) * (kTT + kT), *dinv = D + kTT;
    double v[kT];  // the thread's row of L, or column of U
    if (tid < n1 * kT) {
      // a row of L: x U = v
      double *P = tile_at(k + 1 + (tid >> 4), k) + (tid & 15) * kT;
#pragma unroll
      for (int c = 0; c < kT; c += 2) {
        const double2 p = *reinterpret_cast<const double2 *>(P + c);
        v[c] = p.x;
        v[c + 1] = p.y;
      }
#pragma unroll
      for (int c = 0; c < kT; ++c) {
        v[c] *= dinv[c];
#pragma unroll
        for (int m = c + 1; m < kT; ++m) v[m] = fma(-v[c], D[c * kT + m], v[m]);
      }
      double *to = Lp + (tid >> 4) * kTT + (tid & 15);
#pragma unroll
      for (int c = 0; c < kT; c += 2) {
        *reinterpret_cast<double2 *>(P + c) = make_double2(v[c], v[c + 1]);
        to[c * kT] = v[c];
        to[(c + 1) * kT] = v[c + 1];
      }
    } else if (tid < 2 * n1 * kT) {
      // a column of U: L x = v
      const int q = tid - n1 * kT;
      double *P = tile_at(k, k + 1 + (q >> 4)) + (q & 15);
#pragma unroll
      for (int c = 0; c < kT; ++c) v[c] = P[c * kT];
#pragma unroll
      for (int c = 0; c < kT; ++c)
#pragma unroll
        for (int m = c + 1; m < kT; ++m) v[m] = fma(-D[m * kT + c], v[c], v[m]);
      double *to = Up + (q >> 4) * kTT + (q & 15);
#pragma unroll
      for (int c = 0; c < kT; ++c) {
        P[c * kT] = v[c];
        to[c * kT] = v[c];
      }
    }
    if (wave == NW - 1) {
      // the right-hand side: L x = v, a row per lane (the groups alike)
      double l[kT], y = R[k * kT + l16];
#pragma unroll
      for (int c = 0; c < kT; ++c) l[c] = c < l16 ? D[l16 * kT + c] : 0.0;
      forward_steps<0>(y, l);
      if (lane < kT) R[k * kT + l16] = Y[l16] = y;
    }
    __syncthreads();
    if (tid < n1 * kT) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < kT; ++c) s = fma(v[c], Y[c], s);
      R[(k + 1) * kT + tid] -= s;
    }
    // the rest of the front: tile t of it loses L U
    auto load = [&](int t) {
      const double *C = tile_at(k + 1 + t / n1, k + 1 + t % n1) + lane;
      v4d acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = C[r * 64];
      return acc;
    };
    auto take = [&](int t, v4d acc) {
      const double *l = Lp + (t / n1) * kTT + lane, *u = Up + (t % n1) * kTT + lane;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-l[s * 64], u[s * 64], acc, 0, 0, 0);
      return acc;
    };
    const bool ahead = k + 1 < mt;  // a panel follows
    if (ahead && wave == 0) {
      double *next = Dall + ((k + 1) & 1) * (kTT + kT);
      front_diag(take(0, load(0)), tile_at(k + 1, k + 1), next, next + kTT, nd.ns - (k + 1) * kT, lane);
    } else {
      // kB tiles of a wave at a time
      constexpr int kB = 4;
      const int w = ahead ? wave - 1 : wave, nw = ahead ? NW - 1 : NW, first = ahead ? 1 : 0, n = n1 * n1;
      for (int t0 = first + w; t0 < n; t0 += kB * nw) {
        v4d acc[kB];
#pragma unroll
        for (int b = 0; b < kB; ++b) acc[b] = load(min(t0 + b * nw, n - 1));
#pragma unroll
        for (int b = 0; b < kB; ++b) acc[b] = take(min(t0 + b * nw, n - 1), acc[b]);
#pragma unroll
        for (int b = 0; b < kB; ++b) {
          const int t = t0 + b * nw;
          if (t >= n) break;
          double *C = tile_at(k + 1 + t / n1, k + 1 + t % n1) + lane;
#pragma unroll
          for (int r = 0; r < 4; ++r) C[r * 64] = acc[b][r];
        }
      }
    }
    __syncthreads();
  }
  for (int r = tid; r < nt * kT; r += NW * 64) Rf[r] = R[r];
}

// x_S = U_SS^{-1} (y_S - U_SB x_B) of every node of a tier, into xt (tree
// order) and off the state.  A wave has every NW-th row of tiles: their sums
// (kOwn at most) with the solved columns stay spread over its lanes until the row's turn,
// when it adds them up, solves the diagonal tile (a row per lane) and hands
// the 16 values over in LDS.  What bounds it: that chain, about 0.5 us a tile.
template <int NW, int kOwn>
__global__ __launch_bounds__(NW * 64) void front_back(const double *fronts, const FrontNode *nodes, int32_t node0,
                                                      const int32_t *border, const int32_t *row_x, double *xt,
                                                      double *x) {
  static_assert(kTreeLeafRows <= kLeafWaves * kT && kTreeTopRows <= 2 * kUpperWaves * kT, "rows of tiles");
  __shared__ double X[(kTreeTopRows > kUpperTiles * kT ? kTreeTopRows : kUpperTiles * kT) + kT];
  const FrontNode nd = nodes[node0 + blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = nd.nt, mt = nd.mt;
  const double *F = fronts + nd.f0, *Rf = F + (int64_t)nt * nt * kTT;
  auto tile_at = [&](int i, int j) { return F + (int64_t)(i * nt + j) * kTT; };
  for (int b = tid; b < (nt - mt) * kT; b += NW * 64) X[mt * kT + b] = b < nd.nb ? xt[border[nd.border0 + b]] : 0.0;
  // the wave's diagonal tiles (row l16 right of the diagonal) and y
  double d[kOwn][kT], y[kOwn], rl[kOwn], acc[kOwn][4];
#pragma unroll
  for (int o = 0; o < kOwn; ++o) {
    const int i = wave + o * NW;
    y[o] = rl[o] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[o][q] = 0.0;
#pragma unroll
    for (int c = 0; c < kT; ++c) d[o][c] = 0.0;
    if (i >= mt) continue;
    const double *T = tile_at(i, i) + l16 * kT;
    y[o] = Rf[i * kT + l16];
    double diag = 1.0;
#pragma unroll
    for (int c = 0; c < kT; ++c) {
      const double v = T[c];
      diag = c == l16 ? v : diag;
      d[o][c] = c > l16 ? v : 0.0;
    }
    rl[o] = 1.0 / diag;
  }
  __syncthreads();
  // a row's tile times the 16 values of its column
  auto load = [&](int i, int j, double (&t)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) t[q] = tile_at(i, j)[q * 64 + lane];
  };
#pragma unroll
  for (int o = 0; o < kOwn; ++o) {
    const int i = wave + o * NW;
    if (i >= mt) continue;
    for (int j = mt; j < nt; ++j) {
      double t[4];
      load(i, j, t);
      const double v = X[j * kT + l16];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[o][q] = fma(t[q], v, acc[o][q]);
    }
  }
  // the tiles of the next two columns
  double t[kOwn][4], next[kOwn][4], later[kOwn][4];
  auto prefetch = [&](int k, double (&to)[kOwn][4]) {
#pragma unroll
    for (int o = 0; o < kOwn; ++o)
      if (wave + o * NW < k) load(wave + o * NW, k, to[o]);
  };
  if (mt > 0) prefetch(mt - 1, t);
  if (mt > 1) prefetch(mt - 2, next);
  for (int k = mt - 1; k >= 0; --k) {
    if (k > 1) prefetch(k - 2, later);
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      if (wave + o * NW != k) continue;
      // row 4 q + g of the sums is register q of group g: lane l16 takes row l16
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double a = group_sum(acc[o][q]);
        s = (l16 >> 2) == q ? a : s;
      }
      double v = y[o] - __shfl(s, (l16 & 3) * 16 + l16);
      back_steps<kT - 1>(v, d[o], rl[o]);
      v *= rl[o];
      if (g == 0) {
        X[k * kT + l16] = v;
        if (k * kT + l16 < nd.ns) {
          const int32_t row = nd.row0 + k * kT + l16;
          xt[row] = v;
          x[row_x[row]] -= v;
        }
      }
    }
    __syncthreads();
    const double v = X[k * kT + l16];
#pragma unroll
    for (int o = 0; o < kOwn; ++o)
      if (wave + o * NW < k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[o][q] = fma(t[o][q], v, acc[o][q]);
      }
#pragma unroll
    for (int o = 0; o < kOwn; ++o)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        t[o][q] = next[o][q];
        next[o][q] = later[o][q];
      }
  }
}

__global__ __launch_bounds__(256) void front_clear(double *f, int64_t n) {
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2; i < n; i += (int64_t)gridDim.x * 512) {
    f[i] = 0.0;
    f[i + 1] = 0.0;
  }
}

// Entry e of a tier's fronts: the sum of its sources in their order, entries
// of G_x (~index) and of the fronts below; then the tier's right-hand sides,
// a row of g and what the fronts below left.
struct FrontSums {
  const int32_t *dst, *ptr, *src;     // entries
  const int32_t *rdst, *rptr, *rsrc;  // right-hand sides, by tree position less first
  const int32_t *row_g;
  int32_t first;
};
__global__ __launch_bounds__(256) void front_gather(double *fronts, FrontSums S, int32_t e0, int32_t e1, int32_t r0,
                                                    int32_t r1, const double *gx, const double *g) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  double s = 0.0;
  if (i < e1 - e0) {
    const int32_t e = e0 + i;
    for (int32_t q = S.ptr[e]; q < S.ptr[e + 1]; ++q) {
      const int32_t at = S.src[q];
      s += at < 0 ? gx[~at] : fronts[at];
    }
    fronts[S.dst[e]] = s;
  } else if (i - (e1 - e0) < r1 - r0) {
    const int32_t row = r0 + i - (e1 - e0), e = row - S.first;
    s = g[S.row_g[row]];
    for (int32_t q = S.rptr[e]; q < S.rptr[e + 1]; ++q) s += fronts[S.rsrc[q]];
    fronts[S.rdst[e]] = s;
  }
}

// The pivot test: a pivot below 1e-13 times its row's largest entry of G_x
// (or not finite) marks the row.
struct FrontRow {
  int32_t front, pos, a0, a1;  // the pivot's value and flat position; entries of G_x
};
__global__ __launch_bounds__(256) void front_pivots(const double *fronts, const FrontRow *rows, int32_t n,
                                                    const int32_t *row_src, const double *gx, double *stat) {
  const int32_t e = blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const FrontRow r = rows[e];
  const double d = fronts[r.front];
  double amax = 0.0;
  for (int32_t q = r.a0; q < r.a1; ++q) amax = fmax(amax, fabs(gx[row_src[q]]));
  if (!isfinite(d) || !(fabs(d) > 1e-13 * amax) || amax == 0.0) stat[2] = (double)(e + 1);
}

// The fronts' factors into the flat layout: per entry of the plan one of L
// and one of U, per row its pivot.
__global__ __launch_bounds__(256) void front_out(const double *fronts, const int2 *at, const int32_t *lo,
                                                 const int32_t *up, int32_t n, const FrontRow *rows, int32_t n_rows,
                                                 double *lu) {
  const int32_t e = blockIdx.x * 256 + threadIdx.x;
  if (e < n_rows) lu[rows[e].pos] = fronts[rows[e].front];
  if (e < n) {
    const int2 f = at[e];
    lu[lo[e]] = fronts[f.x];
    lu[up[e]] = fronts[f.y];
  }
}

}  // namespace

struct DevFronts {
  std::vector<void *> allocs;
  int64_t bytes = 0;
  double *fronts = nullptr;
  int64_t leaf_values = 0, values = 0;
  const FrontNode *nodes = nullptr;
  const int32_t *a_dst = nullptr, *a_src = nullptr;  // leaves: entries of G_x
  FrontSums sums{};                                  // the tiers above
  const int32_t *border = nullptr;                   // tree positions
  double *xt = nullptr;                              // the step, in tree order
  const int2 *at = nullptr;                                 // per plan entry: its L and U values in the fronts
  const int32_t *lo = nullptr, *up = nullptr, *row_src = nullptr;
  const FrontRow *rows = nullptr;
  int32_t n = 0, n_ents = 0;
  // per tier: first node, sum and row, most tiles and tiles of own rows of a node
  std::vector<int32_t> tier, ents, rows_at, most, most_own;
};

namespace {

rh_status f_alloc(DevFronts &f, size_t n, void **out, std::string &err) {
  const rh_status s = device_try_alloc(out, n, err);
  if (s != RH_OK) return s;
  f.allocs.push_back(*out);
  f.bytes += (int64_t)n;
  return RH_OK;
}

template <class T>
rh_status f_up(DevFronts &f, const std::vector<T> &v, const T **out, std::string &err) {
  void *p = nullptr;
  const rh_status s = f_alloc(f, std::max<size_t>(sizeof(T), v.size() * sizeof(T)), &p, err);
  if (s != RH_OK) return s;
  if (!v.empty()) HIP_TRY(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  *out = static_cast<const T *>(p);
  return RH_OK;
}

// The fronts of a network may take this much; beyond it (more than a million
// states) the row-by-row factorisation remains.
constexpr int64_t kMostFrontBytes = int64_t(4) << 30;
int64_t front_values(int32_t nt) { return (int64_t)nt * nt * kTT + nt * kT; }

size_t front_lds(int32_t nt) {
  return ((size_t)2 * (nt - 1) * kTT + 2 * (kTT + kT) + kT + nt * kT) * sizeof(double);
}

rh_status fill(DevFronts &f, const LuPlan &lu, const LuMaps &mp, const TreePlan &p, std::string &err) {
  const int32_t n = lu.n, n_nodes = (int32_t)p.nodes.size(), tiers = (int32_t)p.tier.size() - 1;
  f.n = n;
  f.tier = p.tier;
  std::vector<FrontNode> nodes(n_nodes);
  std::vector<int32_t> owner(n);  // tree position -> node
  int64_t total = 0;
  for (int32_t t = 0; t < tiers; ++t) {
    int32_t most = 0, most_own = 0;
    for (int32_t q = p.tier[t]; q < p.tier[t + 1]; ++q) {
      const TreeNode &nd = p.nodes[q];
      nodes[q] = FrontNode{total, nd.ns, nd.nb, nd.mt, nd.mt + nd.bt, 0, 0, nd.row0, nd.border0};
      total += front_values(nodes[q].nt);
      most = std::max(most, nodes[q].nt);
      most_own = std::max(most_own, nd.mt);
      for (int32_t a = 0; a < nd.ns; ++a) owner[nd.row0 + a] = q;
    }
    f.most.push_back(most);
    f.most_own.push_back(most_own);
    if (t == 0) f.leaf_values = total;
  }
  f.values = total;
  // local row of a node in its front's tiles, and the value (r, c)
  auto tiled = [](const TreeNode &nd, int32_t l) { return l < nd.ns ? l : nd.mt * kT + l - nd.ns; };
  auto value = [&](int32_t q, int32_t r, int32_t c) {  // tiled rows
    return nodes[q].f0 + (int64_t)((r / kT) * nodes[q].nt + c / kT) * kTT + (r % kT) * kT + c % kT;
  };
  // G_x by the node that eliminates the earlier of row and column
  struct Entry {
    int32_t r, c, src;  // tree positions
  };
  std::vector<std::vector<Entry>> of_node(n_nodes);
  for (int32_t i = 0; i < n; ++i)
    for (int32_t e = mp.a_ptr[i]; e < mp.a_ptr[i + 1]; ++e) {
      const int32_t r = p.pos[i], c = p.pos[mp.lucol[mp.row_ptr[i] + mp.a_dst[e]]];
      of_node[owner[std::min(r, c)]].push_back({r, c, mp.a_src[e]});
    }
  // the nodes with border rows in a node
  std::vector<std::vector<int32_t>> below(n_nodes);
  for (int32_t q = 0; q < n_nodes; ++q) {
    const TreeNode &nd = p.nodes[q];
    for (int32_t b = 0; b < nd.nb; ++b) {
      auto &v = below[owner[p.border[nd.border0 + b]]];
      if (v.empty() || v.back() != q) v.push_back(q);
    }
  }
  std::vector<int32_t> a_dst, a_src, dst, ptr, src, at(n, -1), loc;
  f.ents.assign(tiers + 1, 0);
  const bool leaves = tiers > 1;  // (a single node is assembled like the upper ones)
  for (int32_t t = 0; t < tiers; ++t) {
    for (int32_t q = p.tier[t]; q < p.tier[t + 1]; ++q) {
      const TreeNode &nd = p.nodes[q];
      for (int32_t a = 0; a < nd.ns; ++a) at[nd.row0 + a] = tiled(nd, a);
      for (int32_t b = 0; b < nd.nb; ++b) at[p.border[nd.border0 + b]] = tiled(nd, nd.ns + b);
      if (t == 0 && leaves) {
        nodes[q].a0 = (int32_t)a_dst.size();
        for (const Entry &e : of_node[q]) {
          a_dst.push_back((int32_t)(value(q, at[e.r], at[e.c]) - nodes[q].f0));
          a_src.push_back(e.src);
        }
        nodes[q].a1 = (int32_t)a_dst.size();
      } else {
        // lists of sources by value, in order
        const int32_t w = nodes[q].nt * kT;
        std::vector<int32_t> head((size_t)w * w, -1), tail((size_t)w * w, -1), next, what;
        auto add = [&](int32_t r, int32_t c, int32_t s) {
          const size_t k = (size_t)r * w + c;
          const int32_t id = (int32_t)what.size();
          what.push_back(s);
          next.push_back(-1);
          (tail[k] >= 0 ? next[tail[k]] : head[k]) = id;
          tail[k] = id;
        };
        for (const Entry &e : of_node[q]) add(at[e.r], at[e.c], ~e.src);
        for (int32_t ch : below[q]) {
          const TreeNode &cd = p.nodes[ch];
          for (int32_t i = 0; i < cd.nb; ++i)
            for (int32_t j = 0; j < cd.nb; ++j) {
              const int32_t r = p.border[cd.border0 + i], c = p.border[cd.border0 + j];
              // (a pair that is not in the front is a zero of the pattern:
              // rows of different subtrees of the node below)
              if (owner[std::min(r, c)] != q || at[r] < 0 || at[c] < 0) continue;
              add(at[r], at[c], (int32_t)value(ch, tiled(cd, cd.ns + i), tiled(cd, cd.ns + j)));
            }
        }
        for (int32_t r = 0; r < w; ++r)
          for (int32_t c = 0; c < w; ++c) {
            int32_t id = head[(size_t)r * w + c];
            if (id < 0) continue;
            dst.push_back((int32_t)value(q, r, c));
            ptr.push_back((int32_t)src.size());
            for (; id >= 0; id = next[id]) src.push_back(what[id]);
          }
      }
      for (int32_t a = 0; a < nd.ns; ++a) at[nd.row0 + a] = -1;
      for (int32_t b = 0; b < nd.nb; ++b) at[p.border[nd.border0 + b]] = -1;
    }
    f.ents[t + 1] = (int32_t)dst.size();
  }
  ptr.push_back((int32_t)src.size());
  // right-hand sides: the rows of g, and above the leaves their sums
  std::vector<int32_t> row_g(n), rdst, rptr, rsrc;
  for (int32_t i = 0; i < n; ++i) row_g[p.pos[i]] = lu.perm[i];
  const int32_t first = leaves ? (p.tier[1] < n_nodes ? p.nodes[p.tier[1]].row0 : n) : 0;
  {
    std::vector<std::vector<int32_t>> left(n - first);
    for (int32_t q = 0; q < n_nodes; ++q) {
      const TreeNode &nd = p.nodes[q];
      const int64_t r0 = nodes[q].f0 + (int64_t)nodes[q].nt * nodes[q].nt * kTT;
      for (int32_t b = 0; b < nd.nb; ++b)
        left[p.border[nd.border0 + b] - first].push_back((int32_t)(r0 + nd.mt * kT + b));
    }
    for (int32_t r = first; r < n; ++r) {
      const FrontNode &nd = nodes[owner[r]];
      rdst.push_back((int32_t)(nd.f0 + (int64_t)nd.nt * nd.nt * kTT + r - nd.row0));
      rptr.push_back((int32_t)rsrc.size());
      rsrc.insert(rsrc.end(), left[r - first].begin(), left[r - first].end());
    }
    rptr.push_back((int32_t)rsrc.size());
  }
  for (int32_t t = 0; t < tiers; ++t)
    f.rows_at.push_back(p.tier[t] < n_nodes ? p.nodes[p.tier[t]].row0 : n);
  f.rows_at.push_back(n);
  f.sums.first = first;
  // the way out
  std::vector<int2> where(p.col.size());
  for (int32_t q = 0; q < n_nodes; ++q) {
    const TreeNode &nd = p.nodes[q];
    for (int32_t a = 0; a < nd.ns + nd.nb; ++a)
      for (int32_t e = p.ent_ptr[nd.ent0 + a]; e < p.ent_ptr[nd.ent0 + a + 1]; ++e) {
        const int32_t r = tiled(nd, a), c = p.col[e];
        where[e] = make_int2((int32_t)value(q, r, c), (int32_t)value(q, c, r));
      }
  }
  std::vector<FrontRow> rows(n);
  for (int32_t i = 0; i < n; ++i) {
    const int32_t q = owner[p.pos[i]], a = p.pos[i] - p.nodes[q].row0;
    rows[i] = FrontRow{(int32_t)value(q, a, a), mp.row_ptr[i] + mp.nl[i], mp.a_ptr[i], mp.a_ptr[i + 1]};
  }
  f.n_ents = (int32_t)where.size();
  rh_status s;
  if ((s = f_up(f, nodes, &f.nodes, err)) != RH_OK || (s = f_up(f, a_dst, &f.a_dst, err)) != RH_OK ||
      (s = f_up(f, a_src, &f.a_src, err)) != RH_OK || (s = f_up(f, dst, &f.sums.dst, err)) != RH_OK ||
      (s = f_up(f, ptr, &f.sums.ptr, err)) != RH_OK || (s = f_up(f, src, &f.sums.src, err)) != RH_OK ||
      (s = f_up(f, rdst, &f.sums.rdst, err)) != RH_OK || (s = f_up(f, rptr, &f.sums.rptr, err)) != RH_OK ||
      (s = f_up(f, rsrc, &f.sums.rsrc, err)) != RH_OK || (s = f_up(f, row_g, &f.sums.row_g, err)) != RH_OK ||
      (s = f_up(f, p.border, &f.border, err)) != RH_OK ||
      (s = f_up(f, where, &f.at, err)) != RH_OK || (s = f_up(f, p.lo, &f.lo, err)) != RH_OK ||
      (s = f_up(f, p.up, &f.up, err)) != RH_OK || (s = f_up(f, rows, &f.rows, err)) != RH_OK ||
      (s = f_up(f, mp.a_src, &f.row_src, err)) != RH_OK)
    return s;
  void *m = nullptr;
  if ((s = f_alloc(f, std::max<size_t>(1, (size_t)f.values) * sizeof(double), &m, err)) != RH_OK) return s;
  f.fronts = static_cast<double *>(m);
  if ((s = f_alloc(f, std::max<size_t>(1, n) * sizeof(double), &m, err)) != RH_OK) return s;
  f.xt = static_cast<double *>(m);
  for (const void *kernel : {reinterpret_cast<const void *>(&front_factor<kLeafWaves, true>),
                             reinterpret_cast<const void *>(&front_factor<kUpperWaves, false>)})
    if ((s = lds_bound(kernel, front_lds(*std::max_element(f.most.begin(), f.most.end())), err)) != RH_OK) return s;
  return RH_OK;
}

}  // namespace

rh_status fronts_build(const LuPlan &lu, const LuMaps &mp, DevFronts **out, std::string &err) {
  *out = nullptr;
  const TreePlan p = tree_plan(lu, mp.row_ptr);
  if (!p.ok) return RH_OK;
  int64_t total = 0;
  for (const TreeNode &nd : p.nodes) total += front_values(nd.mt + nd.bt);
  if (total * (int64_t)sizeof(double) > kMostFrontBytes) return RH_OK;
  std::unique_ptr<DevFronts, void (*)(DevFronts *)> f(new DevFronts(), fronts_free);
  const rh_status s = fill(*f, lu, mp, p, err);
  if (s == RH_ENOMEM) {
    // no memory for them: row by row, as for a network that the plan does not take
    err.clear();
    return RH_OK;
  }
  if (s == RH_OK) *out = f.release();
  return s;
}

void fronts_free(DevFronts *f) {
  if (!f) return;
  for (void *p : f->allocs) (void)hipFree(p);
  delete f;
}

int64_t fronts_bytes(const DevFronts *f) { return f ? f->bytes : 0; }

rh_status fronts_refactor(const DevFronts &f, const FrontIo &io, std::string &err) {
  const int32_t tiers = (int32_t)f.tier.size() - 1;
  const int64_t first = tiers > 1 ? f.leaf_values : 0;
  if (f.values > first)
    hipLaunchKernelGGL(front_clear, dim3((uint32_t)std::min<int64_t>(2048, (f.values - first + 511) / 512)), dim3(256),
                       0, nullptr, f.fronts + first, f.values - first);
  for (int32_t t = 0; t < tiers; ++t) {
    const uint32_t nodes = (uint32_t)(f.tier[t + 1] - f.tier[t]);
    const size_t lds = front_lds(std::max(1, f.most[t]));
    if (t == 0 && tiers > 1) {
      hipLaunchKernelGGL((front_factor<kLeafWaves, true>), dim3(nodes), dim3(kLeafWaves * 64), lds, nullptr, f.fronts,
                         f.nodes, 0, f.a_dst, f.a_src, f.sums.row_g, io.gx, io.g);
      continue;
    }
    const int32_t e0 = f.ents[t], e1 = f.ents[t + 1], r0 = f.rows_at[t], r1 = f.rows_at[t + 1];
    if (e1 - e0 + r1 - r0 > 0)
      hipLaunchKernelGGL(front_gather, dim3((e1 - e0 + r1 - r0 + 255) / 256), dim3(256), 0, nullptr, f.fronts, f.sums, e0,
                         e1, r0, r1, io.gx, io.g);
    hipLaunchKernelGGL((front_factor<kUpperWaves, false>), dim3(nodes), dim3(kUpperWaves * 64), lds, nullptr, f.fronts,
                       f.nodes, f.tier[t], f.a_dst, f.a_src, f.sums.row_g, io.gx, io.g);
  }
  hipLaunchKernelGGL(front_pivots, dim3((f.n + 255) / 256), dim3(256), 0, nullptr, f.fronts, f.rows, f.n, f.row_src,
                     io.gx, io.stat);
  HIP_TRY(hipGetLastError());
  return RH_OK;
}

rh_status fronts_solve(const DevFronts &f, const FrontIo &io, std::string &err) {
  const int32_t tiers = (int32_t)f.tier.size() - 1;
  for (int32_t t = tiers - 1; t >= 0; --t) {
    const uint32_t nodes = (uint32_t)(f.tier[t + 1] - f.tier[t]);
    if (t == 0 && tiers > 1)
      hipLaunchKernelGGL((front_back<kLeafWaves, 1>), dim3(nodes), dim3(kLeafWaves * 64), 0, nullptr, f.fronts, f.nodes, 0,
                         f.border, f.sums.row_g, f.xt, io.x);
    else if (f.most_own[t] <= kUpperWaves)
      hipLaunchKernelGGL((front_back<kUpperWaves, 1>), dim3(nodes), dim3(kUpperWaves * 64), 0, nullptr, f.fronts, f.nodes,
                         f.tier[t], f.border, f.sums.row_g, f.xt, io.x);
    else
      hipLaunchKernelGGL((front_back<kUpperWaves, 2>), dim3(nodes), dim3(kUpperWaves * 64), 0, nullptr, f.fronts, f.nodes,
                         f.tier[t], f.border, f.sums.row_g, f.xt, io.x);
  }
  HIP_TRY(hipGetLastError());
  return RH_OK;
}

rh_status fronts_factors(const DevFronts &f, const FrontIo &io, std::string &err) {
  hipLaunchKernelGGL(front_out, dim3((std::max(f.n_ents, f.n) + 255) / 256), dim3(256), 0, nullptr, f.fronts, f.at,
                     f.lo, f.up, f.n_ents, f.rows, f.n, io.lu);
  HIP_TRY(hipGetLastError());
  return RH_OK;
}

}  // namespace rh
