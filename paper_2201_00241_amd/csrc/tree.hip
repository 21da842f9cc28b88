// Kernels of the tree path: Algorithm 2 for many directions on the nodes of
// tree.cpp's plan.
//
// The path that keeps a direction in one workgroup (device.hip) streams all
// of a network's factor records once per direction, and a launch takes as
// long as one direction's chain of dependent steps (280 us at 10k buses, 16 ms
// at 70k, where the vector lies in global memory), however few directions
// there are.  Here a sweep is a few launches of small dense products: a node's
// triangle is applied as its explicit inverse (at most 448 rows, in tiles of
// 16), 16 directions to a matrix instruction, so that a node has no chain but
// the sums themselves, the nodes of a tier are spread over the chip, and a
// leaf's matrices are read once for all the chunks of 16 directions that its
// workgroup takes.
//
// One call is a fixed sequence of launches on the caller's stream: tier by
// tier forward and backward for Z, the projection, the same for Psi, and the
// assembly.  A direction's arithmetic depends on the network alone, not on k,
// its place in a chunk, or the launch it shares.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <type_traits>

#include "tree.h"
#include "tree_device.h"

namespace rh {

namespace {

#define AS4 __attribute__((address_space(4)))
#define HIP_TRY(expr)                                                          \
  do {                                                                         \
    hipError_t e_ = (expr);                                                    \
    if (e_ != hipSuccess) {                                                    \
      err = std::string(#expr) + ": " + hipGetErrorString(e_);                 \
      return RH_EDEVICE;                                                       \
    }                                                                          \
  } while (0)

constexpr int kD = kTreeDirs, kT = kTreeTile;
static_assert(kD == 16 && kT == 16, "the shape of the matrix instructions");
constexpr int kTileVals = kT * kT;  // a tile in operand order: value [s][lane] is entry
                                    // (lane mod 16, 4 s + lane / 16)
// Workgroups a tier's launch has at most where a node has several chunks to
// take: what the chip holds at once, twice over.
constexpr uint32_t kLeafGroups = 2048, kProjGroups = 8192, kResGroups = 1024;
// Chunks a workgroup takes in turn at most (it keeps a bit for each).
constexpr int32_t kChunkRun = 64;
// Dynamic LDS of a workgroup: 160 KB less the little that is static.
constexpr size_t kTreeLds = 159 * 1024;

typedef double v4d __attribute__((ext_vector_type(4)));

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Row of output register q of a lane in group g = lane / 16.
__device__ __forceinline__ int mfma_row(int q, int g) { return 4 * q + g; }

// The refined mode: the leaves multiply and sum in FP64, with the FP64
// matrices; FP32 sums there left the results twice as far from exact as the
// substitutions of the one-workgroup path.  Above the leaves FP64 gains nothing
// more: the matrices are FP32, and so is an output tile's sum, in four parts
// (one per four columns of the tiles) that need not wait for each other.
template <class T>
struct UpperTile;
template <>
struct UpperTile<double> {
  v4d a;
  __device__ __forceinline__ void clear() { a = v4d{0.0, 0.0, 0.0, 0.0}; }
  __device__ __forceinline__ void take(int, double m, double x) { a = mfma16(m, x, a); }
  __device__ __forceinline__ v4d sum() const { return a; }
  static __device__ __forceinline__ int row(int q, int g) { return mfma_row(q, g); }
};
template <>
struct UpperTile<float> {
  v4f a[4];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  }
  __device__ __forceinline__ void take(int s, float m, float x) {
    a[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(m, x, a[s], 0, 0, 0);
  }
  __device__ __forceinline__ v4f sum() const { return (a[0] + a[1]) + (a[2] + a[3]); }
  static __device__ __forceinline__ int row(int q, int g) { return 4 * g + q; }  // (a group's rows together)
};

// Lane J of each group of 16 lanes to all its lanes.
template <int J>
__device__ __forceinline__ int row_bcast(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + J, 0xF, 0xF, true);
}
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + J, 0xF, 0xF, true);
}

// LDS-only barrier: workgroups exchange data through LDS, so that loads in
// flight (the matrices') stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A pointer that is the same in all lanes, in scalar registers: what it points
// to is then read by the scalar unit, in one trip.
template <class P>
__device__ __forceinline__ P *uniform(P *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<P *>((uint64_t)hi << 32 | lo);
}

// Item of a chunk (items sorted by their first).
__device__ __forceinline__ TreeItem item_of(const TreeArgs &a, int32_t chunk) {
  if (!a.items) return a.one;
  const TreeItem AS4 *items = (const TreeItem AS4 *)a.items;
  int32_t lo = 0, hi = a.n_items - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (items[mid].chunk0 <= chunk)
      lo = mid;
    else
      hi = mid - 1;
  }
  const TreeItem AS4 &s = items[__builtin_amdgcn_readfirstlane(lo)];
  TreeItem it;
  it.td = s.td;
  it.W = s.W;
  it.HW = s.HW;
  it.ldw = s.ldw;
  it.ldhw = s.ldhw;
  it.k = s.k;
  it.identity_from = s.identity_from;
  it.chunk0 = s.chunk0;
  it.chunks = s.chunks;
  it.at = s.at;
  it.stride = s.stride;
  it.rinfo = s.rinfo;
  return it;
}
__device__ __forceinline__ const TreeDesc AS4 &desc_of(const TreeItem &it) {
  return *(const TreeDesc AS4 *)uniform(it.td);
}

// A chunk's memory in the launch scratch, rows of kD values, as byte offsets:
// directions, Y_p, state, second solve, update rows.  Refined mode: in the
// place of the update rows the FP32 correction and its update rows.
struct ChunkOff {
  uint32_t W, P, Z, Y, U;
};
constexpr uint32_t kRow64 = kD * sizeof(double), kRow32 = kD * sizeof(float);
__device__ __forceinline__ ChunkOff chunk_off(const TreeDesc AS4 &td) {
  ChunkOff o;
  o.W = 0;
  o.P = (uint32_t)td.n_p * kRow64;
  o.Z = 2 * o.P;
  o.Y = o.Z + (uint32_t)td.n_x * kRow64;
  o.U = o.Y + (uint32_t)td.n_x * kRow64;
  return o;
}
template <class T>
__device__ __forceinline__ uint32_t upd_off(const TreeDesc AS4 &td, const ChunkOff &o) {
  return sizeof(T) == 8 ? o.U : o.U + (uint32_t)td.n_x * kRow32;
}

// Reads and writes of a chunk's memory go through a buffer descriptor of
// exactly that memory: an offset past its end (kNone) reads zero and writes
// nothing, so rows that are not there cost no branch, and the loads of a
// chunk can be counted past the stores of the one before.
typedef unsigned v2u __attribute__((ext_vector_type(2)));
constexpr uint32_t kNone = 0x80000000u;
struct ChunkBuf {
  __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ double *chunk_mem(const TreeArgs &a, const TreeItem &it, int32_t chunk) {
  return a.scratch + (int64_t)(it.at + chunk * it.stride) * kTreeLine;
}
__device__ __forceinline__ ChunkBuf chunk_buf(const TreeArgs &a, const TreeItem &it, int32_t chunk) {
  return ChunkBuf{__builtin_amdgcn_make_buffer_rsrc(chunk_mem(a, it, chunk), 0,
                                                    it.stride * kTreeLine * (int)sizeof(double), 0x00027000)};
}
template <class S>
__device__ __forceinline__ S get(const ChunkBuf &m, uint32_t off) {
  if constexpr (sizeof(S) == 8)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(m.r, off, 0, 0));
  else
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(m.r, off, 0, 0));
}
__device__ __forceinline__ void put(const ChunkBuf &m, uint32_t off, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), m.r, off, 0, 0);
}
__device__ __forceinline__ void put(const ChunkBuf &m, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), m.r, off, 0, 0);
}

// w of parameter q in the lane's direction (chunk column dir of the item).
__device__ __forceinline__ double w_of(const TreeItem &it, const ChunkBuf &m, int32_t q, int32_t dir, int l16) {
  if (it.identity_from >= 0) return (q == it.identity_from + dir && dir < it.k) ? 1.0 : 0.0;
  return get<double>(m, (uint32_t)q * kRow64 + (uint32_t)l16 * 8);
}

// Refined mode: {max |r|, max |x|} of a chunk's directions after iteration
// `iter` of solve `which` (0: Z, 1: Psi).  Zero for a direction that took no
// correction in it.
__device__ __forceinline__ const double *norms_at(const TreeArgs &a, int32_t chunk, int which, int iter) {
  return a.norms + (((int64_t)chunk * 2 + which) * a.norm_iters + iter) * 2 * kD;
}
// Whether direction l16 of the chunk still takes corrections in iteration
// `iter`: the iteration before left it a residual above the tolerance (one
// that had stopped earlier has zero norms there, and zero is not above zero).
__device__ __forceinline__ bool still_active(const TreeArgs &a, const TreeDesc AS4 &td, int32_t chunk, int which,
                                             int iter, int l16) {
  if (iter == 0) return true;
  const double *nm = norms_at(a, chunk, which, iter - 1);
  return !(nm[l16] <= a.tol * ((which ? td.norm_t : td.norm_n) * nm[kD + l16]));
}
// Bit c: whether chunk first + c has such directions, up to chunk end - 1 (at
// most kChunkRun of them); the same in every lane.  Four chunks a trip.
__device__ __forceinline__ uint64_t active_chunks(const TreeArgs &a, const TreeDesc AS4 &td, int32_t first, int32_t end,
                                                  int which, int iter) {
  if (iter == 0) return ~uint64_t(0);
  const int lane = threadIdx.x & 63;
  uint64_t active = 0;
  for (int32_t c = 0; c < end - first; c += 4) {
    const int32_t chunk = first + c + (lane >> 4);
    const uint64_t b = __ballot(chunk < end && still_active(a, td, min(chunk, end - 1), which, iter, lane & 15));
    for (int g = 0; g < 4; ++g) active |= (uint64_t)((b >> (16 * g) & 0xffff) != 0) << (c + g);
  }
  return active;
}

// The matrices of sweep `s` (0: L, 1: U, 2: U^T, 3: L^T) in operand order, from
// product p0 of its list on.
template <class T>
__device__ __forceinline__ const T *sweep_mat(const TreeDesc AS4 &td, int s, int32_t p0);
template <>
__device__ __forceinline__ const double *sweep_mat<double>(const TreeDesc AS4 &td, int s, int32_t p0) {
  return td.m64[s] + (int64_t)p0 * kTileVals;
}
template <>
__device__ __forceinline__ const float *sweep_mat<float>(const TreeDesc AS4 &td, int s, int32_t p0) {
  return td.m32[s] + (int64_t)(p0 - td.first32[s & 1]) * kTileVals;
}

// Sums over N sparse rows of val * x(col), x giving a column's value in the
// lane's direction.  A row's first 16 entries are loaded one per lane of the
// group and broadcast; the rows' pointers, entries and first AT columns'
// values are each requested for all rows before any is waited for, as a trip
// to memory costs more than all else here.
template <int N>
struct SparseRows {
  int32_t e[N], n[N], c[N];
  double v[N];
};
// row(j): the j-th row, or -1
template <int N, class R>
__device__ __forceinline__ void rows_load(SparseRows<N> &s, const int32_t *ptr, const int32_t *col, const double *val,
                                          int l16, R row) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const uint32_t r = (uint32_t)max(row(j), 0);
    s.e[j] = ptr[r];
    s.n[j] = ptr[r + 1];
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    s.n[j] = row(j) < 0 ? 0 : s.n[j] - s.e[j];
    s.c[j] = 0;
    s.v[j] = 0.0;
    if (l16 < s.n[j]) {
      s.c[j] = col[(uint32_t)(s.e[j] + l16)];
      s.v[j] = val[(uint32_t)(s.e[j] + l16)];
    }
  }
}
// acc += entries J.. of the n <= 16 in the group's lanes, four in flight.
template <int J, class F>
__device__ __forceinline__ void row_rest(double &acc, double v, int32_t c, int n, F x) {
  if constexpr (J < 16) {
    if (J < n) {
      double w[4];
      w[0] = x(row_bcast<J>(c));
      w[1] = J + 1 < 16 ? x(row_bcast<(J + 1) & 15>(c)) : 0.0;
      w[2] = J + 2 < 16 ? x(row_bcast<(J + 2) & 15>(c)) : 0.0;
      w[3] = J + 3 < 16 ? x(row_bcast<(J + 3) & 15>(c)) : 0.0;
      acc = fma(row_bcast<J>(v), w[0], acc);
      if (J + 1 < n) acc = fma(row_bcast<(J + 1) & 15>(v), w[1], acc);
      if (J + 2 < n) acc = fma(row_bcast<(J + 2) & 15>(v), w[2], acc);
      if (J + 3 < n) acc = fma(row_bcast<(J + 3) & 15>(v), w[3], acc);
      row_rest<J + 4>(acc, v, c, n, x);
    }
  }
}
template <int J, int AT, class W, class F>
__device__ __forceinline__ void row_first(W (&w)[AT], int32_t c, int n, F x) {
  if constexpr (J < AT) {
    w[J] = W(0);
    if (J < n) w[J] = x(row_bcast<J>(c));
    row_first<J + 1, AT, W>(w, c, n, x);
  }
}
template <int J, int AT, class W>
__device__ __forceinline__ void row_fma(double &acc, const W (&w)[AT], double v, int n) {
  if constexpr (J < AT) {
    if (J < n) acc = fma(row_bcast<J>(v), (double)w[J], acc);
    row_fma<J + 1, AT, W>(acc, w, v, n);
  }
}
// The same for columns whose values lie at base + bytes * column in a chunk's
// memory (S: their type; l16: added per lane): every row's first AT loads are
// issued without a test, those past the row's end reading zero (kNone), so
// that nothing but the sum depends on the rows' lengths.  rows_at turns the
// columns into offsets.
template <int N>
__device__ __forceinline__ void rows_at(SparseRows<N> &s, uint32_t base, uint32_t bytes, int l16) {
#pragma unroll
  for (int j = 0; j < N; ++j) s.c[j] = (int32_t)(l16 < s.n[j] ? base + (uint32_t)s.c[j] * bytes : kNone);
}
template <int J, int AT, class S>
__device__ __forceinline__ void row_values(S (&w)[AT], int32_t c, const ChunkBuf &m, uint32_t lane_off) {
  if constexpr (J < AT) {
    w[J] = get<S>(m, (uint32_t)row_bcast<J>(c) + lane_off);
    row_values<J + 1, AT, S>(w, c, m, lane_off);
  }
}
template <int J, int AT, class S>
__device__ __forceinline__ void row_dot(double &acc, const S (&w)[AT], double v) {
  if constexpr (J < AT) {
    acc = fma(row_bcast<J>(v), (double)w[J], acc);
    row_dot<J + 1, AT, S>(acc, w, v);
  }
}
template <int AT, class S, int N>
__device__ __forceinline__ void rows_sum_at(const SparseRows<N> &s, const int32_t *col, const double *val, uint32_t base,
                                            uint32_t bytes, const ChunkBuf &m, int l16, double (&acc)[N]) {
  const uint32_t lane_off = (uint32_t)l16 * (uint32_t)sizeof(S);
  S w[N][AT];
#pragma unroll
  for (int j = 0; j < N; ++j) row_values<0, AT, S>(w[j], s.c[j], m, lane_off);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    acc[j] = 0.0;
    row_dot<0, AT, S>(acc[j], w[j], s.v[j]);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if (s.n[j] <= AT) continue;
    row_rest<AT>(acc[j], s.v[j], s.c[j], min(16, s.n[j]), [&](int32_t o) { return get<S>(m, (uint32_t)o + lane_off); });
    for (int32_t e = 16; e < s.n[j]; ++e) {
      const int32_t at = s.e[j] + e;
      acc[j] = fma(val[at], (double)get<S>(m, base + (uint32_t)col[at] * bytes + lane_off), acc[j]);
    }
  }
}

template <int AT, int N, class F>
__device__ __forceinline__ void rows_sum(const SparseRows<N> &s, const int32_t *col, const double *val, int l16, F x,
                                         double (&acc)[N]) {
  typedef decltype(x(0)) W;
  W w[N][AT];
#pragma unroll
  for (int j = 0; j < N; ++j) row_first<0, AT, W>(w[j], s.c[j], s.n[j], x);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    acc[j] = 0.0;
    row_fma<0, AT, W>(acc[j], w[j], s.v[j], s.n[j]);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if (s.n[j] <= AT) continue;
    if constexpr (AT >= 4) {
      row_rest<AT>(acc[j], s.v[j], s.c[j], min(16, s.n[j]), x);
    } else {  // (seldom, and a loop takes fewer registers)
      for (int e = AT; e < min(16, s.n[j]); ++e) acc[j] = fma(__shfl(s.v[j], e, 16), x(__shfl(s.c[j], e, 16)), acc[j]);
    }
    for (int32_t e = 16; e < s.n[j]; e += 16) {
      const int n = min(16, s.n[j] - e);
      const int32_t at = s.e[j] + e + (l16 < n ? l16 : 0);  // lanes past the row repeat an entry, unused
      const int32_t c = col[at];
      const double v = val[at];
      for (int q = 0; q < n; ++q) acc[j] = fma(__shfl(v, q, 16), x(__shfl(c, q, 16)), acc[j]);
    }
  }
}

// ---- nodes --------------------------------------------------------------

// The records of N rows above the leaves (-1: none), and the sum of the
// update rows (at byte offset upd) they receive, added to v; all rows' values
// in flight together.
struct Gat {
  int32_t g[kTreeGat];
};
template <int N>
__device__ __forceinline__ void gat_load(const TreeDesc AS4 &td, const int32_t (&row)[N], Gat (&g)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int4 *p = td.gat + (uint32_t)(max(row[j], td.gat0) - td.gat0) * (kTreeGat / 4);
#pragma unroll
    for (int q = 0; q < kTreeGat / 4; ++q) {
      const int4 r = p[q];
      g[j].g[4 * q] = r.x;
      g[j].g[4 * q + 1] = r.y;
      g[j].g[4 * q + 2] = r.z;
      g[j].g[4 * q + 3] = r.w;
    }
  }
}
template <class T, int N>
__device__ __forceinline__ void add_updates(const TreeDesc AS4 &td, const int32_t (&row)[N], const Gat (&g)[N],
                                            const ChunkBuf &m, uint32_t upd, int l16, T (&v)[N]) {
  auto at = [&](int32_t r) { return get<T>(m, r >= 0 ? upd + (uint32_t)(r * kD + l16) * (uint32_t)sizeof(T) : kNone); };
  T u[N][4];
#pragma unroll
  for (int h = 0; h < kTreeGat; h += 4) {
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) u[j][q] = at(row[j] >= 0 ? g[j].g[h + q] : -1);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += (u[j][0] + u[j][1]) + (u[j][2] + u[j][3]);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int32_t list = row[j] >= 0 ? g[j].g[kTreeGat - 1] : -1;
    if (list > -2) continue;
    const int32_t *more = td.gat_more - 2 - list;
    const int32_t n = more[0];
    for (int32_t e = 0; e < n; e += 8) {
      T w[8];
#pragma unroll
      for (int h = 0; h < 8; ++h) w[h] = at(e + h < n ? more[1 + e + h] : -1);
#pragma unroll
      for (int h = 0; h < 8; ++h) v[j] += w[h];
    }
  }
}

template <class T>
__device__ __forceinline__ void tile_load(const T *mat, int32_t p, int lane, T (&a)[4]) {
  const T *t = mat + (int64_t)p * kTileVals + lane;
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = t[s * 64];
}
// The first RING matrix tiles of n products (mat: their first).
template <class T, int RING>
__device__ __forceinline__ void ring_start(const T *mat, int32_t n, int lane, T (&H)[RING][4]) {
#pragma unroll
  for (int h = 0; h < RING; ++h)
    if (h < n) tile_load<T>(mat, h, lane, H[h]);
}

// A wave's n products (ents: the list, one per lane; mat: their matrix tiles): sums of
// matrix tiles times input tiles of X (LDS, rows of kD), out(r, acc) per
// finished output tile; done() once H is free.  H is a ring of the matrix tiles
// in flight, its first ones loaded.  An output tile may span waves: the later ones leave their
// sums in `parts` (LDS, a tile per wave), and after a barrier the first adds
// them in their order.
template <class T, int RING, class G, class F>
__device__ __forceinline__ void products(T (&H)[RING][4], int32_t ents, int32_t n, const T *mat, const T *X,
                                         T *parts, int wave, int lane, G done, F out) {
  const T *Xl = X + (lane >> 4) * kD + (lane & 15);
  UpperTile<T> acc;
  acc.clear();
  int32_t more = 0, last = 0;
  for (int32_t p = 0; p < n; p += RING) {
#pragma unroll
    for (int h = 0; h < RING; ++h) {
      if (p + h >= n) break;
      const int32_t e = __builtin_amdgcn_readlane(ents, p + h);
      const T *x = Xl + (e & kProdMask) * (kT * kD);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc.take(s, H[h][s], x[4 * s * kD]);
      if (e & kProdLast) {
        more = e >> kProdMore;
        if (more) {  // (the wave's last product)
          last = e;
          break;
        }
        const auto v = acc.sum();
        if (e & kProdPart) {
#pragma unroll
          for (int q = 0; q < 4; ++q) parts[(wave * 4 + q) * 64 + lane] = v[q];
        } else {
          out((e >> kProdBits) & kProdMask, v);
        }
        acc.clear();
      }
      if (p + h + RING < n) tile_load<T>(mat, p + h + RING, lane, H[h]);
    }
  }
  done();
  lds_barrier();
  if (more) {
    auto v = acc.sum();
    for (int w = wave + 1; w <= wave + more; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += parts[(w * 4 + q) * 64 + lane];
    out((last >> kProdBits) & kProdMask, v);
  }
}

// Matrix tiles in flight per wave above the leaves.
constexpr int kRing = 4;
// Rows a lane group stages: the node's own (forward), or its border's too.
constexpr int kStageFwd = 4, kLeafStage = 6, kUpperStage = 8;
static_assert(kLeafTiles * kT <= kLeafStage * kLeafWaves * 4 && kUpperTiles * kT <= kUpperStage * kUpperWaves * 4 &&
                  kTreeLeafRows <= kStageFwd * kLeafWaves * 4 && kTreeUpperRows <= kStageFwd * kUpperWaves * 4,
              "staging");

// What a solve's sweeps read and write.  SP: the first forward sweep in FP64,
// whose right-hand side B = -P G_p W is formed on the way.  Refined (T =
// float): the forward sweep reads the FP64 residual, and what is solved for
// is the FP32 correction.
template <class T, bool FWD>
struct SweepIo {
  static constexpr bool kRef = sizeof(T) == 4;
  typedef typename std::conditional<kRef && !FWD, float, double>::type S;  // a staged row's type
  static __device__ __forceinline__ uint32_t in(const ChunkOff &o, int which) {
    return kRef && !FWD ? o.U : which == 0 && !kRef ? o.Z : o.Y;
  }
  static __device__ __forceinline__ uint32_t out(const ChunkOff &o, int which) {
    return kRef ? o.U : which == 0 ? o.Z : o.Y;
  }
};

// Byte offset of the lane's value of row i of M's tiles where its products go:
// the node's own rows, or (forward) the update rows of its border.
template <class T, bool FWD>
__device__ __forceinline__ uint32_t out_off(const TreeNode AS4 &nd, int32_t i, uint32_t own, uint32_t upd, int l16) {
  const int32_t b = i - nd.mt * kT;
  const uint32_t o = own + (uint32_t)((nd.row0 + i) * kD + l16) * (uint32_t)sizeof(T);
  const uint32_t u = upd + (uint32_t)((nd.u0 + b) * kD + l16) * (uint32_t)sizeof(T);
  return i < nd.ns ? o : FWD && b >= 0 && b < nd.nb ? u : kNone;
}

// One leaf, the chunks blockIdx.y * per .. + per - 1 in turn.  FWD: M b_S, b_S
// the right-hand side; the solution's rows replace it and the border's update
// rows go up.  Else M^T [ D^{-1} y_S ; x_B ], in place.
//
// A leaf's matrices stay in its waves' registers from chunk to chunk (at most
// six tiles and two output tiles a wave, so that all loops are unrolled and a
// chunk's loads and stores have no branches), and a chunk costs its own rows:
// in, one barrier (the staging buffer in LDS is double), the products, and
// out; the next chunk's rows are requested before the products.  With many
// chunks the tier is bound by those rows' traffic, with few by the launch and
// the trips to memory.
template <class T, bool FWD, bool SP>
__global__ __launch_bounds__(kLeafWaves * 64, 4) void tree_leaf(const TreeArgs a, int which, int iter, int per) {
  extern __shared__ __align__(16) char lds_raw[];
  typedef SweepIo<T, FWD> Io;
  typedef typename Io::S S;
  constexpr bool kRef = Io::kRef;
  constexpr int kSlots = kLeafWaves * 4, kStage = FWD ? kStageFwd : kLeafStage;
  const int tid = threadIdx.x, slot = tid >> 4, l16 = tid & 15, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (a.stamps && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0 && FWD && iter == 0)
    a.stamps[which == 0 ? 1 : 4] = wall_clock64();
  const int32_t c1 = min((int32_t)blockIdx.y * per + per, a.n_chunks);
  int buf = 0;
  for (int32_t chunk = (int32_t)blockIdx.y * per; chunk < c1;) {
    const TreeItem it = item_of(a, chunk);
    const TreeDesc AS4 &td = desc_of(it);
    const int32_t end = min(c1, it.chunk0 + it.chunks);
    uint64_t active = kRef ? active_chunks(a, td, chunk, end, which, iter) : ~uint64_t(0);
    if (td.n_tiers < 2 || (int32_t)blockIdx.x >= td.tier[1] || !active) {  // no such leaf in this network
      chunk = end;
      continue;
    }
    const TreeNode AS4 &nd = *(const TreeNode AS4 *)(td.nodes + blockIdx.x);
    const uint16_t AS4 *wave_at = FWD ? nd.fwd_at : nd.bwd_at;
    const int32_t np = wave_at[wave + 1] - wave_at[wave], p0 = (FWD ? nd.fwd0 : nd.bwd0) + wave_at[wave];
    const int32_t ns = nd.ns, mt = nd.mt, rows = (FWD ? mt : mt + nd.bt) * kT;
    const ChunkOff off = chunk_off(td);
    const int32_t ents = lane < np ? (FWD ? td.fwd : td.bwd)[p0 + lane] : 0;
    double H[kLeafProds][4];
    ring_start(sweep_mat<double>(td, which == 0 ? (FWD ? 0 : 1) : (FWD ? 2 : 3), p0), np, lane, H);
    // where the staged rows are
    uint32_t at[kStage];
    SparseRows<SP ? kStageFwd : 1> gp;
#pragma unroll
    for (int j = 0; j < kStage; ++j) {
      const int32_t r = slot + j * kSlots, b = r - mt * kT;
      int32_t row = r < ns ? nd.row0 + r : -1;
      if constexpr (!FWD) {
        const bool in = b >= 0 && b < nd.nb;
        const int32_t br = td.border[nd.border0 + (in ? b : 0)];
        row = in ? br : row;
      }
      at[j] = row >= 0 ? Io::in(off, which) + (uint32_t)(row * kD + l16) * (uint32_t)sizeof(S) : kNone;
    }
    if constexpr (SP)
      rows_load(gp, td.gp_ptr, td.gp_col, td.gp_val, l16,
                [&](int j) { return slot + j * kSlots < ns ? nd.row0 + slot + j * kSlots : -1; });
    // the wave's products: inputs, and the output tiles' places
    int32_t in[kLeafProds], n0 = 0;
    uint32_t to[2][4];
#pragma unroll
    for (int h = kLeafProds - 1; h >= 0; --h) {
      const int32_t e = __builtin_amdgcn_readlane(ents, h);
      in[h] = (e & kProdMask) * (kT * kD);
      if (h < np && (e & kProdLast)) n0 = h + 1;
    }
    const int32_t e0 = __builtin_amdgcn_readlane(ents, n0 > 0 ? n0 - 1 : 0);
    const int32_t e1 = __builtin_amdgcn_readlane(ents, np > n0 ? np - 1 : 0);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int32_t r = ((o ? e1 : e0) >> kProdBits) & kProdMask;
      const bool used = o ? np > n0 : n0 > 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        to[o][q] = used ? out_off<T, FWD>(nd, r * kT + mfma_row(q, lane >> 4), Io::out(off, which),
                                          upd_off<T>(td, off), l16)
                        : kNone;
    }
    S v[kStage];
    if constexpr (!SP) {
      const ChunkBuf m = chunk_buf(a, it, chunk);
#pragma unroll
      for (int j = 0; j < kStage; ++j) v[j] = get<S>(m, at[j]);
      // As many stores (to nowhere) as a chunk's follow its loads in the loop:
      // with the same count on both ways in, the wait for the loads leaves the
      // stores in flight.
#pragma unroll
      for (int o = 0; o < 8; ++o) put(m, kNone, T(0));
    }
    for (; chunk < end; ++chunk, active >>= 1) {
      const ChunkBuf m = chunk_buf(a, it, chunk);
      double *X = reinterpret_cast<double *>(lds_raw) + buf * a.lds_rows * kD;
      buf ^= 1;
      double x[kStage];
      if constexpr (SP) {
        const int32_t dir = (chunk - it.chunk0) * kD + l16;
        double b[kStageFwd];
        rows_sum<2>(gp, td.gp_col, td.gp_val, l16, [&](int32_t q) { return w_of(it, m, q, dir, l16); }, b);
#pragma unroll
        for (int j = 0; j < kStageFwd; ++j) x[j] = -b[j];
      } else {
#pragma unroll
        for (int j = 0; j < kStage; ++j) x[j] = (double)v[j];
      }
#pragma unroll
      for (int j = 0; j < kStage; ++j)
        if (slot + j * kSlots < rows) X[(slot + j * kSlots) * kD + l16] = x[j];
      lds_barrier();
      if constexpr (!SP) {
        const ChunkBuf next = chunk_buf(a, it, min(chunk + 1, end - 1));
#pragma unroll
        for (int j = 0; j < kStage; ++j) v[j] = get<S>(next, at[j]);
      }
      const bool skip = kRef && !(active & 1);
      const double *Xl = X + (lane >> 4) * kD + l16;
      v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int h = 0; h < kLeafProds; ++h) {
        if (h >= np || skip) break;
        double xs[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) xs[s] = Xl[in[h] + 4 * s * kD];
        if (h < n0) {
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[0] = mfma16(H[h][s], xs[s], acc[0]);
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[1] = mfma16(H[h][s], xs[s], acc[1]);
        }
      }
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q) put(m, skip ? kNone : to[o][q], (T)acc[o][q]);
    }
  }
}

// One node above the leaves and one chunk: as tree_leaf, the right-hand side
// with the updates of the nodes below, and the matrices read as they come up.
template <class T, bool FWD, bool SP>
__global__ __launch_bounds__(kUpperWaves * 64, 4) void tree_upper(const TreeArgs a, int tier, int which, int iter) {
  extern __shared__ __align__(16) char lds_raw[];
  typedef SweepIo<T, FWD> Io;
  typedef typename Io::S S;
  constexpr bool kRef = Io::kRef;
  constexpr int kSlots = kUpperWaves * 4, kStage = FWD ? kStageFwd : kUpperStage;
  const int tid = threadIdx.x, slot = tid >> 4, l16 = tid & 15, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t chunk = blockIdx.y;
  const TreeItem it = item_of(a, chunk);
  const TreeDesc AS4 &td = desc_of(it);
  if (tier >= td.n_tiers - 1) return;
  const int32_t node = td.tier[tier] + (int32_t)blockIdx.x;
  if (node >= td.tier[tier + 1]) return;
  if (kRef && !__any(still_active(a, td, chunk, which, iter, l16))) return;
  const TreeNode AS4 &nd = *(const TreeNode AS4 *)(td.nodes + node);
  const uint16_t AS4 *wave_at = FWD ? nd.fwd_at : nd.bwd_at;
  const int32_t np = wave_at[wave + 1] - wave_at[wave], p0 = (FWD ? nd.fwd0 : nd.bwd0) + wave_at[wave];
  const int32_t ns = nd.ns, mt = nd.mt, rows = (FWD ? mt : mt + nd.bt) * kT;
  const ChunkOff off = chunk_off(td);
  const ChunkBuf m = chunk_buf(a, it, chunk);
  const int32_t ents = lane < np ? (FWD ? td.fwd : td.bwd)[p0 + lane] : 0;
  const T *mat = sweep_mat<T>(td, which == 0 ? (FWD ? 0 : 1) : (FWD ? 2 : 3), p0);
  T x[kStage];
  T H[kRing][4];
  ring_start(mat, np, lane, H);
  Gat g[kStageFwd];
  int32_t row[kStage];
#pragma unroll
  for (int j = 0; j < kStage; ++j) {
    const int32_t r = slot + j * kSlots, b = r - mt * kT;
    row[j] = r < ns ? nd.row0 + r : -1;
    if constexpr (!FWD) {
      const bool in = b >= 0 && b < nd.nb;
      const int32_t br = td.border[nd.border0 + (in ? b : 0)];
      row[j] = in ? br : row[j];
    }
  }
  if constexpr (FWD) gat_load(td, row, g);
  if constexpr (SP) {
    const int32_t dir = (chunk - it.chunk0) * kD + l16;
    SparseRows<kStageFwd> gp;
    rows_load(gp, td.gp_ptr, td.gp_col, td.gp_val, l16, [&](int j) { return row[j]; });
    double b[kStageFwd];
    rows_sum<2>(gp, td.gp_col, td.gp_val, l16, [&](int32_t q) { return w_of(it, m, q, dir, l16); }, b);
#pragma unroll
    for (int j = 0; j < kStageFwd; ++j) x[j] = (T)-b[j];
  } else {
    const uint32_t src = Io::in(off, which);
#pragma unroll
    for (int j = 0; j < kStage; ++j)
      x[j] = (T)get<S>(m, row[j] >= 0 ? src + (uint32_t)(row[j] * kD + l16) * (uint32_t)sizeof(S) : kNone);
  }
  if constexpr (FWD) add_updates<T>(td, row, g, m, upd_off<T>(td, off), l16, x);
  T *X = reinterpret_cast<T *>(lds_raw);
#pragma unroll
  for (int j = 0; j < kStage; ++j)
    if (slot + j * kSlots < rows) X[(slot + j * kSlots) * kD + l16] = x[j];
  lds_barrier();
  const uint32_t own = Io::out(off, which), upd = upd_off<T>(td, off);
  products(H, ents, np, mat, X, X + a.lds_rows * kD, wave, lane, [] {}, [&](int32_t r, const auto &acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      put(m, out_off<T, FWD>(nd, r * kT + UpperTile<T>::row(q, lane >> 4), own, upd, l16), (T)acc[q]);
  });
}

// The top node of a chunk: forward, D^{-1}, backward, its vector in LDS
// throughout.
template <class T, bool SP>
__global__ __launch_bounds__(kUpperWaves * 64, 4) void tree_top(const TreeArgs a, int which, int iter) {
  extern __shared__ __align__(16) char lds_raw[];
  constexpr bool kRef = sizeof(T) == 4;
  constexpr int kSlots = kUpperWaves * 4;
  const int tid = threadIdx.x, slot = tid >> 4, l16 = tid & 15, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t chunk = blockIdx.x;
  const TreeItem it = item_of(a, chunk);
  const TreeDesc AS4 &td = desc_of(it);
  if (a.stamps && chunk == 0 && tid == 0 && td.n_tiers == 1 && iter == 0) a.stamps[which == 0 ? 1 : 4] = wall_clock64();
  if (kRef && !__any(still_active(a, td, chunk, which, iter, l16))) return;
  const TreeNode AS4 &nd = *(const TreeNode AS4 *)(td.nodes + td.tier[td.n_tiers - 1]);
  const ChunkOff off = chunk_off(td);
  const ChunkBuf m = chunk_buf(a, it, chunk);
  const int32_t ns = nd.ns, mt = nd.mt, row0 = nd.row0, dir = (chunk - it.chunk0) * kD + l16;
  T *X = reinterpret_cast<T *>(lds_raw), *X2 = X + mt * kT * kD;
  T *parts = X2 + mt * kT * kD;
  const int32_t np = nd.fwd_at[wave + 1] - nd.fwd_at[wave], p0 = nd.fwd0 + nd.fwd_at[wave];
  const int32_t nq = nd.bwd_at[wave + 1] - nd.bwd_at[wave], q0 = nd.bwd0 + nd.bwd_at[wave];
  const int32_t ents = lane < np ? td.fwd[p0 + lane] : 0, ents2 = lane < nq ? td.bwd[q0 + lane] : 0;
  T H[kRing][4];
  const T *mat = sweep_mat<T>(td, which == 0 ? 0 : 2, p0), *mat2 = sweep_mat<T>(td, which == 0 ? 1 : 3, q0);
  if constexpr (!SP) ring_start(mat, np, lane, H);
  const uint32_t src = SweepIo<T, true>::in(off, which), own = SweepIo<T, true>::out(off, which);
  for (int32_t r0 = slot; r0 < mt * kT; r0 += 4 * kSlots) {
    T v[4];
    Gat g[4];
    int32_t row[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) row[j] = r0 + j * kSlots < ns ? row0 + r0 + j * kSlots : -1;
    gat_load(td, row, g);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (!SP)
        v[j] = (T)get<double>(m, row[j] >= 0 ? src + (uint32_t)(row[j] * kD + l16) * 8u : kNone);
    }
    if constexpr (SP) {
      SparseRows<4> gp;
      rows_load(gp, td.gp_ptr, td.gp_col, td.gp_val, l16, [&](int j) { return row[j]; });
      rows_sum<2>(gp, td.gp_col, td.gp_val, l16, [&](int32_t q) { return w_of(it, m, q, dir, l16); }, v);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = -v[j];
    }
    add_updates<T>(td, row, g, m, upd_off<T>(td, off), l16, v);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int32_t r = r0 + j * kSlots;
      if (r >= mt * kT) break;
      X[r * kD + l16] = v[j];
    }
  }
  if constexpr (SP) ring_start(mat, np, lane, H);  // (the registers are taken before)
  lds_barrier();
  auto second = [&] { ring_start(mat2, nq, lane, H); };
  products(H, ents, np, mat, X, parts, wave, lane, second, [&](int32_t r, const auto &acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q) X2[(r * kT + UpperTile<T>::row(q, lane >> 4)) * kD + l16] = (T)acc[q];
  });
  lds_barrier();
  if (a.stamps && chunk == 0 && tid == 0) a.stamps[which == 0 ? 2 : 5] = wall_clock64();
  products(H, ents2, nq, mat2, X2, parts, wave, lane, [] {}, [&](int32_t r, const auto &acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      put(m, out_off<T, false>(nd, r * kT + UpperTile<T>::row(q, lane >> 4), own, 0, l16), (T)acc[q]);
  });
}

// ---- directions in, projection, products out ----------------------------------

// The chunk's directions in rows of kD (W transposed through LDS: 64
// parameters at a time, so that both sides are whole lines); columns past
// the item's k are zero.  The refined mode also clears its norms and
// forms B = -P G_p W here for the rows without entries.
constexpr int kMoveRows = 64;
__global__ __launch_bounds__(256) void tree_in(const TreeArgs a) {
  __shared__ double s[kMoveRows][kD + 1];
  const int32_t chunk = blockIdx.y;
  const TreeItem it = item_of(a, chunk);
  const TreeDesc AS4 &td = desc_of(it);
  double *mem = chunk_mem(a, it, chunk);
  const int tid = threadIdx.x;
  if (a.stamps && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) a.stamps[0] = wall_clock64();
  if (a.norms) {
    // refined mode: clear the norms and the right-hand side
    if (blockIdx.x == 0) {
      double *nm = const_cast<double *>(norms_at(a, chunk, 0, 0));
      for (int32_t i = tid; i < 4 * a.norm_iters * kD; i += 256) nm[i] = 0.0;
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < (int64_t)td.n_x * kD; i += (int64_t)gridDim.x * 256)
      mem[chunk_off(td).Y / 8 + i] = 0.0;
  }
  if (it.identity_from >= 0) return;
  const int32_t d0 = (chunk - it.chunk0) * kD;
  for (int32_t q0 = blockIdx.x * kMoveRows; q0 < td.n_p; q0 += gridDim.x * kMoveRows) {
    for (int32_t e = tid; e < kMoveRows * kD; e += 256) {
      const int32_t q = e % kMoveRows, d = e / kMoveRows;
      s[q][d] = q0 + q < td.n_p && d0 + d < it.k ? it.W[(int64_t)(d0 + d) * it.ldw + q0 + q] : 0.0;
    }
    __syncthreads();
    for (int32_t e = tid; e < kMoveRows * kD; e += 256) {
      const int32_t q = e / kD, d = e % kD;
      if (q0 + q < td.n_p) mem[(int64_t)(q0 + q) * kD + d] = s[q][d];
    }
    __syncthreads();
  }
}

// Refined mode: the rows of B = -P G_p W with entries.
__global__ __launch_bounds__(256) void tree_spmul(const TreeArgs a) {
  const int32_t chunk = blockIdx.y;
  const TreeItem it = item_of(a, chunk);
  const TreeDesc AS4 &td = desc_of(it);
  const ChunkBuf m = chunk_buf(a, it, chunk);
  const uint32_t y = chunk_off(td).Y;
  const int slot = threadIdx.x >> 4, l16 = threadIdx.x & 15;
  const int32_t dir = (chunk - it.chunk0) * kD + l16;
  for (int32_t g = blockIdx.x * 16 + slot; g < td.n_gp_rows; g += gridDim.x * 16) {
    const int4 r = td.gp_rows[g];
    SparseRows<1> s;
    double acc[1];
    rows_load(s, &td.gp_rows[g].y, td.gp_col, td.gp_val, l16, [](int) { return 0; });
    rows_sum<4>(s, td.gp_col, td.gp_val, l16, [&](int32_t q) { return w_of(it, m, q, dir, l16); }, acc);
    put(m, y + (uint32_t)(r.x * kD + l16) * 8u, -acc[0]);
  }
}

// Tensor projection: 16 lanes per bus, its incidences in turn.  -Y_x into Y,
// the voltage parameters' Y_p into P.
constexpr int kProjBuses = 16;  // buses per workgroup: one per lane group
constexpr int kProjInc = 4;     // incidences whose loads are in flight together
__global__ __launch_bounds__(256) void tree_project(const TreeArgs a, int per) {
  const int tid = threadIdx.x, l16 = tid & 15;
  // consecutive buses on the workgroups of one XCD: neighbours' rows are in its L2
  const int32_t b = ((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * kProjBuses + (tid >> 4);
  if (a.stamps && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) a.stamps[3] = wall_clock64();
  const int32_t c1 = min((int32_t)blockIdx.y * per + per, a.n_chunks);
  for (int32_t chunk = (int32_t)blockIdx.y * per; chunk < c1;) {
    const TreeItem it = item_of(a, chunk);
    const TreeDesc AS4 &td = desc_of(it);
    const int32_t end = min(c1, it.chunk0 + it.chunks);
    if (b >= td.n_bus) {
      chunk = end;
      continue;
    }
    const TreeBus B = td.bus[b];
    const int32_t ni = B.inc1 - B.inc0;
    TreeInc I[kProjInc];
#pragma unroll
    for (int j = 0; j < kProjInc; ++j)
      if (j < ni) I[j] = td.inc[B.inc0 + j];
    const ChunkOff off = chunk_off(td);
    const bool id = it.identity_from >= 0;
    // the buses' angle and voltage: a state, or the parameter's direction
    auto theta_at = [&](int32_t tx) { return tx >= 0 ? off.Z + (uint32_t)(tx * kD + l16) * 8u : kNone; };
    auto volt_at = [&](int32_t vs) {
      return vs >= 0 ? off.Z + (uint32_t)(vs * kD + l16) * 8u : id ? kNone : (uint32_t)((-vs - 1) * kD + l16) * 8u;
    };
    uint32_t ot[kProjInc], ov[kProjInc];
#pragma unroll
    for (int j = 0; j < kProjInc; ++j) {
      ot[j] = j < ni ? theta_at(I[j].ot) : kNone;
      ov[j] = j < ni ? volt_at(I[j].ov) : kNone;
    }
    const uint32_t bt = theta_at(B.tx), bv = volt_at(B.vs);
    const uint32_t yt = B.tx >= 0 ? off.Y + (uint32_t)(B.tx * kD + l16) * 8u : kNone;
    const uint32_t yv_at = B.vs >= 0 ? off.Y + (uint32_t)(B.vs * kD + l16) * 8u
                                     : off.P + (uint32_t)((-B.vs - 1) * kD + l16) * 8u;
    for (; chunk < end; ++chunk) {
      const ChunkBuf m = chunk_buf(a, it, chunk);
      const int32_t dir = (chunk - it.chunk0) * kD + l16;
      // identity directions are not stored
      auto one = [&](double v, int32_t vs) {
        return id && vs < 0 && -vs - 1 == it.identity_from + dir && dir < it.k ? 1.0 : v;
      };
      double to[kProjInc], vo[kProjInc];
      const double dte = get<double>(m, bt);
      double dve = get<double>(m, bv);
#pragma unroll
      for (int j = 0; j < kProjInc; ++j) {
        to[j] = vo[j] = 0.0;
        if (j >= ni) continue;
        to[j] = get<double>(m, ot[j]);
        vo[j] = get<double>(m, ov[j]);
      }
      dve = one(dve, B.vs);
      double yth = 0.0, yv = 0.0;
      if (B.sth != 0.0 || B.sv != 0.0) {
        // the slack-cost rank-one term: only the buses next to the reference
        double sl = 0.0;
        for (int32_t q = 0; q < td.n_slack; ++q) {
          const int2 x = td.slack_x[q];
          const double2 g = td.slack_g[q];
          sl += g.x * get<double>(m, theta_at(x.x)) + g.y * one(get<double>(m, volt_at(x.y)), x.y);
        }
        yth = B.sth * sl;
        yv = B.sv * sl;
      }
      auto add = [&](const TreeInc &in, double t, double v) {
        const double dd = dte - t;
        yth += -in.K * dd + in.Hps * (in.vo * dve + B.ve * v);
        yv += in.Hps * in.vo * dd + in.A2 * dve + in.H * v;
      };
#pragma unroll
      for (int j = 0; j < kProjInc; ++j)
        if (j < ni) add(I[j], to[j], one(vo[j], I[j].ov));
      for (int32_t e = kProjInc; e < ni; ++e) {
        const TreeInc in = td.inc[B.inc0 + e];
        add(in, get<double>(m, theta_at(in.ot)), one(get<double>(m, volt_at(in.ov)), in.ov));
      }
      put(m, yt, -yth);
      put(m, yv_at, B.vs >= 0 ? -yv : yv);
    }
  }
}

// H W = Y_p + G_p^T Psi: a row group per parameter, the tile transposed
// through LDS so that each direction's products leave in whole lines.
__global__ __launch_bounds__(256) void tree_out(const TreeArgs a) {
  __shared__ double s[kMoveRows][kD + 1];
  const int32_t chunk = blockIdx.y;
  const TreeItem it = item_of(a, chunk);
  const TreeDesc AS4 &td = desc_of(it);
  const int32_t q0 = blockIdx.x * kMoveRows;
  if (q0 >= td.n_p) return;
  const ChunkBuf m = chunk_buf(a, it, chunk);
  const ChunkOff off = chunk_off(td);
  const int tid = threadIdx.x, slot = tid >> 4, l16 = tid & 15;
  const int32_t d0 = (chunk - it.chunk0) * kD, dir = d0 + l16;
  if (a.stamps && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) a.stamps[6] = wall_clock64();
  const uint32_t psi = a.norms ? off.Z : off.Y;  // the refined solution, or the solve in place
  constexpr int kRows = kMoveRows / 16;
  auto par = [&](int j) { return q0 + slot + j * 16 < td.n_p ? q0 + slot + j * 16 : -1; };
  double c2[kRows], p[kRows], w[kRows], acc[kRows];
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const int32_t q = max(par(j), 0);
    c2[j] = td.p_c2x2[q];
    p[j] = get<double>(m, off.P + (uint32_t)(q * kD + l16) * 8u);
    w[j] = w_of(it, m, q, dir, l16);
  }
  SparseRows<kRows> gt;
  rows_load(gt, td.gpt_ptr, td.gpt_row, td.gpt_val, l16, par);
  rows_at(gt, psi, kRow64, l16);
  rows_sum_at<8, double>(gt, td.gpt_row, td.gpt_val, psi, kRow64, m, l16, acc);
#pragma unroll
  for (int j = 0; j < kRows; ++j) s[slot + j * 16][l16] = (__builtin_isnan(c2[j]) ? p[j] : __dmul_rn(c2[j], w[j])) + acc[j];
  __syncthreads();
  for (int32_t e = tid; e < kMoveRows * kD; e += 256) {
    const int32_t q = e % kMoveRows, d = e / kMoveRows;
    if (q0 + q < td.n_p && d0 + d < it.k) it.HW[(int64_t)(d0 + d) * it.ldhw + q0 + q] = s[q][d];
  }
  if (a.norms && it.rinfo && blockIdx.x == 0 && tid < kD && dir < it.k) {
    // per-column figures of both solves: the last iteration taken
    double *o = it.rinfo + 4 * (int64_t)dir;
    for (int w = 0; w < 2; ++w) {
      const double an = w ? td.norm_t : td.norm_n;
      double berr = 0.0;
      int steps = 0;
      for (int i = 0; i < a.norm_iters; ++i) {
        const double *nm = norms_at(a, chunk, w, i);
        const double r = nm[l16], sc = an * nm[kD + l16];
        berr = r == 0.0 ? 0.0 : r / sc;
        steps = i;
        if (r <= a.tol * sc) break;
      }
      o[2 * w] = berr;
      o[2 * w + 1] = (double)steps;
    }
  }
  if (a.stamps && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) a.stamps[7] = wall_clock64();
}

// Refined mode: x += d and r -= A d for the directions that still take
// corrections (d the FP32 correction just solved for, x in Z, r in Y, both
// FP64), and the norms max |r|, max |x| of the iteration (non-negative
// doubles compare as their bits).
//
// A workgroup takes its rows for several chunks in turn, so that the rows'
// entries are read once, and stops at once where none of them takes a
// correction (the norms of four chunks are read in one trip).  Bound by the
// chunks' traffic: 16 chunks at 10k buses move 133 MB (171 from the second
// iteration on) in 39 to 47 us, 53 with a chunk per workgroup; with nothing to
// do a launch takes 4 us, 10 before.
constexpr int kResRows = 64, kResAt = 8;
__global__ __launch_bounds__(512) void tree_residual(const TreeArgs a, int which, int iter, int per) {
  __shared__ double s_m[2][8][2][kD];
  const int tid = threadIdx.x, slot = tid >> 4, l16 = tid & 15, wave = tid >> 6;
  const int32_t r0 = blockIdx.x * kResRows;
  const int32_t c1 = min((int32_t)blockIdx.y * per + per, a.n_chunks);
  int buf = 0;
  for (int32_t chunk = (int32_t)blockIdx.y * per; chunk < c1;) {
    const TreeItem it = item_of(a, chunk);
    const TreeDesc AS4 &td = desc_of(it);
    const int32_t end = min(c1, it.chunk0 + it.chunks);
    const uint64_t active = active_chunks(a, td, chunk, end, which, iter);
    if (r0 >= td.n_x || !active) {
      chunk = end;
      continue;
    }
    const ChunkOff off = chunk_off(td);
    const int32_t *ptr = which ? td.at_ptr : td.an_ptr, *col = which ? td.at_col : td.an_col;
    const double *val = which ? td.at_val : td.an_val;
    constexpr int kRows = kResRows / 32;
    auto row = [&](int j) { return r0 + slot + j * 32 < td.n_x ? r0 + slot + j * 32 : -1; };
    SparseRows<kRows> s;
    rows_load(s, ptr, col, val, l16, row);
    rows_at(s, off.U, kRow32, l16);
    const int32_t first = chunk;
    for (; chunk < end; ++chunk) {
      if (!(active >> (chunk - first) & 1)) continue;
      const bool act = still_active(a, td, chunk, which, iter, l16);
      const ChunkBuf m = chunk_buf(a, it, chunk);
      double y[kRows], z[kRows], acc[kRows], rm = 0.0, xm = 0.0;
      float d[kRows];
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const uint32_t at = (uint32_t)(row(j) * kD + l16);
        y[j] = get<double>(m, row(j) < 0 ? kNone : off.Y + at * 8u);
        z[j] = get<double>(m, row(j) < 0 || iter == 0 ? kNone : off.Z + at * 8u);
        d[j] = get<float>(m, row(j) < 0 ? kNone : off.U + at * 4u);
      }
      rows_sum_at<kResAt, float>(s, col, val, off.U, kRow32, m, l16, acc);
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        if (!act || row(j) < 0) continue;
        const uint32_t at = (uint32_t)(row(j) * kD + l16);
        const double r = y[j] - acc[j], x = z[j] + (double)d[j];
        put(m, off.Y + at * 8u, r);
        put(m, off.Z + at * 8u, x);
        rm = fmax(rm, fabs(r));
        xm = fmax(xm, fabs(x));
      }
      for (int o = 16; o <= 32; o <<= 1) {
        rm = fmax(rm, __shfl_xor(rm, o));
        xm = fmax(xm, __shfl_xor(xm, o));
      }
      if ((tid & 63) < kD) {
        s_m[buf][wave][0][l16] = rm;
        s_m[buf][wave][1][l16] = xm;
      }
      __syncthreads();  // (the buffer after the next is this one again: one barrier is enough)
      if (tid < 2 * kD && act) {
        const int w = tid >> 4;
        double v = 0.0;
        for (int q = 0; q < 8; ++q) v = fmax(v, s_m[buf][q][w][l16]);
        double *nm = const_cast<double *>(norms_at(a, chunk, which, iter)) + w * kD + l16;
        atomicMax(reinterpret_cast<unsigned long long *>(nm), (unsigned long long)__double_as_longlong(v));
      }
      buf ^= 1;
    }
  }
}

// ---- values of an operating point ---------------------------------------------

// The entries of the nodes' triangles from the flat factors: L(i, j), and the
// unit factor's U^T(i, j) = U(j, i) / U(j, j).
__global__ __launch_bounds__(256) void tree_fill(const double *f, const int32_t *lo, const int32_t *up,
                                                 const int32_t *dg, int32_t n, double *vl, double *vu) {
  const int32_t e = blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  vl[e] = f[lo[e]];
  vu[e] = f[up[e]] / f[dg[e]];
}

// A sum of two doubles, kept unevaluated.
struct Pair {
  double h, l;
};
__device__ __forceinline__ Pair pair_add(Pair a, Pair b) {
  const double s = a.h + b.h, t = s - a.h;
  return Pair{s, (a.h - (s - t)) + (b.h - t) + a.l + b.l};
}

// Column tile `cols[block].y` of node `cols[block].x`'s matrix, for L (grid y
// 0) and U^T (1): one wave, a column per lane of a group of 16, the four
// groups sharing a row's entries.  Row by row, y_a = (a == j) - sum of
// v(a, c) y_c, with y and the sums as pairs of doubles (products exact by
// FMA, two-sums) and rounded at the end, so that the matrix is as good as one
// formed in extended precision.  Rows of y live in LDS.  Both operand orders
// are written (M for the forward sweep, M^T for the backward one), in FP64
// and from node node32 (above the leaves) on in FP32, whose lists start at
// products first32.x and first32.y.  A row is a chain of LDS reads, so the next row's entries are
// loaded meanwhile.
__global__ __launch_bounds__(64) void tree_invert(const TreeNode *nodes, const int2 *cols, const int32_t *ent_ptr,
                                                  const uint16_t *col, const double *vl, const double *vu,
                                                  const int2 *map, const double *f, const int32_t *dpos, double *fl,
                                                  double *fu, double *bl, double *bu, int32_t node32, int2 first32,
                                                  float *fl32, float *fu32, float *bl32, float *bu32) {
  extern __shared__ __align__(16) char lds_raw[];
  const int2 w = cols[blockIdx.x];
  const TreeNode nd = nodes[w.x];
  const bool upper = blockIdx.y != 0;
  const double *val = upper ? vu : vl;
  const int lane = threadIdx.x, g = lane >> 4, l16 = lane & 15;
  const int32_t rows = nd.ns + nd.nb, a0 = w.y * kT;
  double *Yh = reinterpret_cast<double *>(lds_raw), *Yl = Yh + (int64_t)rows * kD;
  for (int32_t i = lane; i < a0 * kD; i += 64) Yh[i] = Yl[i] = 0.0;
  __syncthreads();
  const int32_t *ptr = ent_ptr + nd.ent0;
  constexpr int kAhead = 4;  // entries per group loaded a row ahead
  int32_t e0 = ptr[a0], e1 = ptr[a0 + 1];
  double v[kAhead];
  int32_t c[kAhead];
  auto load = [&](int32_t from, int32_t to) {
#pragma unroll
    for (int h = 0; h < kAhead; ++h) {
      const int32_t e = from + g + 4 * h;
      v[h] = e < to ? val[e] : 0.0;
      c[h] = e < to ? (int32_t)col[e] : 0;
    }
  };
  load(e0, e1);
  for (int32_t i = a0; i < rows; ++i) {
    Pair s{0.0, 0.0};
    auto take = [&](double x, int32_t at) {
      const double yh = Yh[at * kD + l16], yl = Yl[at * kD + l16];
      const double p = -x * yh;
      s = pair_add(s, Pair{p, fma(-x, yh, -p) - x * yl});
    };
    const int32_t from = e0, to = e1;
    double vc[kAhead];
    int32_t cc[kAhead];
#pragma unroll
    for (int h = 0; h < kAhead; ++h) {
      vc[h] = v[h];
      cc[h] = c[h];
    }
    if (i + 1 < rows) {
      e0 = e1;
      e1 = ptr[i + 2];
      load(e0, e1);
    }
#pragma unroll
    for (int h = 0; h < kAhead; ++h)
      if (from + g + 4 * h < to) take(vc[h], cc[h]);
    for (int32_t e = from + g + 4 * kAhead; e < to; e += 4) take(val[e], col[e]);
    s = pair_add(s, Pair{__shfl_xor(s.h, 16), __shfl_xor(s.l, 16)});
    s = pair_add(s, Pair{__shfl_xor(s.h, 32), __shfl_xor(s.l, 32)});
    if (i == a0 + l16) s = pair_add(s, Pair{1.0, 0.0});
    if (g == 0) {
      const double h = s.h + s.l;
      Yh[i * kD + l16] = h;
      Yl[i * kD + l16] = s.l - (h - s.h);
    }
    __syncthreads();
  }
  double *fo = upper ? fu : fl, *bo = upper ? bu : bl;
  float *fo32 = upper ? fu32 : fl32, *bo32 = upper ? bu32 : bl32;
  for (int32_t r = 0; r < nd.mt + nd.bt; ++r) {
    const int2 t = map[nd.map0 + r * nd.mt + w.y];
    if (t.x < 0) continue;
    // row i of the tile: own rows, or border rows
    const int32_t first = r < nd.mt ? r * kT : nd.ns + (r - nd.mt) * kT;
    const int32_t last = r < nd.mt ? nd.ns : rows;
    auto at = [&](int32_t i, int32_t j) {  // entry (i, j) of the tile; rows above the column are zero
      return first + i < last && a0 + j < nd.ns ? Yh[(first + i) * kD + j] : 0.0;
    };
    const bool own = r < nd.mt && first + l16 < last;
    const double piv = own ? f[dpos[nd.row0 + first + l16]] : 1.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double y = at(4 * s + g, l16);
      double x = at(l16, 4 * s + g);
      if (own && a0 + 4 * s + g < nd.ns) {  // the forward matrix takes the pivots as well
        const double q = x / piv;
        x = q + (fma(-q, piv, x) + Yl[(first + l16) * kD + 4 * s + g]) / piv;
      }
      const int64_t at_f = (int64_t)t.x * kTileVals + s * 64 + lane, b = (int64_t)t.y * kTileVals + s * 64 + lane;
      fo[at_f] = x;
      bo[b] = y;
      if (w.x >= node32) {
        fo32[at_f - (int64_t)first32.x * kTileVals] = (float)x;
        bo32[b - (int64_t)first32.y * kTileVals] = (float)y;
      }
    }
  }
}

__global__ __launch_bounds__(256) void tree_gather(const double *in, const int32_t *src, int32_t n, double *out) {
  const int32_t e = blockIdx.x * 256 + threadIdx.x;
  if (e < n) out[e] = in[src[e]];
}

}  // namespace

// ---- host side --------------------------------------------------------------

struct DevTree {
  int device = -1;
  TreePlan plan;  // its large arrays are freed once uploaded
  std::vector<void *> allocs;
  int64_t bytes = 0;
  TreeDesc d{};
  TreeDesc *dd = nullptr;
  // device arrays that the values of an operating point are formed with
  double *f = nullptr, *gxv = nullptr, *vl = nullptr, *vu = nullptr;
  const int32_t *lo = nullptr, *up = nullptr, *dg = nullptr, *dpos = nullptr, *ent_ptr = nullptr;
  const uint16_t *col = nullptr;
  const int2 *cols = nullptr, *map = nullptr;
  const int32_t *an_src = nullptr, *at_src = nullptr;
  int32_t n_ents = 0, n_cols = 0, nnz_gx = 0, node32 = 0;
  size_t n_flat = 0;
  std::vector<int32_t> row_ptr, bus_order, gp_src, gpt_src;
};

namespace {

template <class T>
rh_status t_alloc(DevTree &t, size_t n, T **out, std::string &err) {
  void *p = nullptr;
  const size_t nb = std::max<size_t>(16, n * sizeof(T));
  const rh_status s = device_try_alloc(&p, nb, err);
  if (s != RH_OK) return s;
  t.allocs.push_back(p);
  t.bytes += (int64_t)nb;
  *out = static_cast<T *>(p);
  return RH_OK;
}

template <class T, class S>
rh_status t_up(DevTree &t, const std::vector<S> &v, const T **out, std::string &err) {
  T *p = nullptr;
  const size_t n = v.size() * sizeof(S);
  rh_status s = t_alloc(t, (n + sizeof(T) - 1) / sizeof(T), &p, err);
  if (s != RH_OK) return s;
  if (n) HIP_TRY(hipMemcpy(p, v.data(), n, hipMemcpyHostToDevice));
  *out = p;
  return RH_OK;
}

#define T_TRY(expr)             \
  do {                          \
    rh_status s_ = (expr);      \
    if (s_ != RH_OK) return s_; \
  } while (0)

// Scratch of one chunk, the larger of the two precisions (FP64 vectors and
// update rows, or FP64 residual and solution with an FP32 correction and 17
// iterations' norms): a network must fit the allocation-free entry point's
// array with one chunk.
int64_t tree_chunk_bytes(int64_t n_x, int64_t n_u, int64_t n_p) {
  return (3 * n_x + n_u + 2 * n_p + 72) * kD * (int64_t)sizeof(double);
}

// Pattern arrays: once per network.
rh_status tree_build(Network &net, DevTree &t, std::string &err) {
  const LuPlan &lu = net.lu;
  const int32_t n = lu.n;
  t.row_ptr.assign(n + 1, 0);
  for (int32_t i = 0; i < n; ++i)
    t.row_ptr[i + 1] = t.row_ptr[i] + (int32_t)(lu.lrow[i].size() + lu.urow[i].size());
  t.n_flat = (size_t)t.row_ptr[n];
  t.plan = tree_plan(lu, t.row_ptr);
  TreePlan &p = t.plan;
  if (!p.ok || (int32_t)p.tier.size() > kTreeTiers ||
      tree_chunk_bytes(lu.n, p.n_u, net.n_p) > (int64_t)RH_NOALLOC_SCRATCH_BYTES) {
    p = TreePlan();
    return RH_OK;
  }
  TreeDesc &d = t.d;
  d.n_x = n;
  d.n_p = net.n_p;
  d.n_bus = net.n_bus;
  d.n_u = p.n_u;
  d.n_tiers = (int32_t)p.tier.size() - 1;
  d.gat0 = p.gat0;
  for (size_t q = 0; q < p.tier.size(); ++q) d.tier[q] = p.tier[q];
  // G_p by tree row
  std::vector<int32_t> order(n);  // tree position -> x index
  for (int32_t i = 0; i < n; ++i) order[p.pos[i]] = lu.perm[i];
  std::vector<int4> grows;
  std::vector<int32_t> gcol;
  std::vector<int32_t> gptr(n + 1, 0);
  for (int32_t r = 0; r < n; ++r) {
    const int32_t x = order[r], e0 = (int32_t)gcol.size();
    for (int32_t e = net.gp.ptr[x]; e < net.gp.ptr[x + 1]; ++e) {
      gcol.push_back(net.gp.col[e]);
      t.gp_src.push_back(e);
    }
    gptr[r + 1] = (int32_t)gcol.size();
    if (gptr[r + 1] > e0) grows.push_back(make_int4(r, e0, gptr[r + 1], 0));
  }
  T_TRY(t_up(t, gptr, &d.gp_ptr, err));
  d.n_gp_rows = (int32_t)grows.size();
  T_TRY(t_up(t, grows, &d.gp_rows, err));
  T_TRY(t_up(t, gcol, &d.gp_col, err));
  // G_p^T: rows in tree order within a parameter
  {
    std::vector<int32_t> ptr(net.n_p + 1, 0), row(gcol.size());
    t.gpt_src.assign(gcol.size(), 0);
    for (int32_t c : gcol) ptr[c + 1]++;
    for (int32_t q = 0; q < net.n_p; ++q) ptr[q + 1] += ptr[q];
    std::vector<int32_t> fill(ptr.begin(), ptr.end() - 1);
    for (const int4 &g : grows)
      for (int32_t e = g.y; e < g.z; ++e) {
        const int32_t k = fill[gcol[e]]++;
        row[k] = g.x;
        t.gpt_src[k] = t.gp_src[e];
      }
    T_TRY(t_up(t, ptr, &d.gpt_ptr, err));
    T_TRY(t_up(t, row, &d.gpt_row, err));
  }
  std::vector<double> c2(net.n_p, std::numeric_limits<double>::quiet_NaN());
  for (int32_t b : net.pv) c2[net.pg_p[b]] = 2.0 * net.c2[net.gen_of_bus[b]];
  T_TRY(t_up(t, c2, &d.p_c2x2, err));
  // buses in tree order of their first state, so that neighbours share nodes
  {
    std::vector<std::pair<int32_t, int32_t>> key(net.n_bus);
    for (int32_t b = 0; b < net.n_bus; ++b)
      key[b] = {net.th_x[b] >= 0 ? p.pos[lu.iperm[net.th_x[b]]] : n, b};
    std::sort(key.begin(), key.end());
    for (auto &k : key) t.bus_order.push_back(k.second);
  }
  T_TRY(t_up(t, p.nodes, &d.nodes, err));
  p.border.push_back(0);  // (a node without border reads the entry at its place)
  T_TRY(t_up(t, p.border, &d.border, err));
  T_TRY(t_up(t, p.gat, &d.gat, err));
  T_TRY(t_up(t, p.gat_more, &d.gat_more, err));
  T_TRY(t_up(t, p.fwd, &d.fwd, err));
  T_TRY(t_up(t, p.bwd, &d.bwd, err));
  T_TRY(t_up(t, p.map, &t.map, err));
  T_TRY(t_up(t, p.ent_ptr, &t.ent_ptr, err));
  T_TRY(t_up(t, p.col, &t.col, err));
  T_TRY(t_up(t, p.lo, &t.lo, err));
  T_TRY(t_up(t, p.up, &t.up, err));
  T_TRY(t_up(t, p.dg, &t.dg, err));
  T_TRY(t_up(t, p.cols, &t.cols, err));
  t.n_ents = (int32_t)p.col.size();
  t.n_cols = (int32_t)p.cols.size() / 2;
  T_TRY(t_alloc(t, p.col.size(), &t.vl, err));
  T_TRY(t_alloc(t, p.col.size(), &t.vu, err));
  const size_t p_fwd = p.fwd.size(), p_bwd = p.bwd.size();
  t.node32 = d.n_tiers > 1 ? p.tier[1] : 0;  // (the leaves are FP64 in both modes)
  d.first32[0] = p.nodes[t.node32].fwd0;
  d.first32[1] = p.nodes[t.node32].bwd0;
  for (int q = 0; q < 4; ++q) {
    double *m = nullptr;
    float *m32 = nullptr;
    const size_t products = q & 1 ? p_bwd : p_fwd;
    T_TRY(t_alloc(t, products * kTileVals, &m, err));
    T_TRY(t_alloc(t, (products - d.first32[q & 1]) * kTileVals, &m32, err));
    d.m64[q] = m;
    d.m32[q] = m32;
  }
  for (std::vector<int32_t> *v : {&p.fwd, &p.bwd, &p.map, &p.ent_ptr, &p.lo, &p.up, &p.dg,
                                  &p.cols, &p.border, &p.gat, &p.gat_more})
    *v = std::vector<int32_t>();
  p.col = std::vector<uint16_t>();
  std::vector<int32_t> dpos(n);
  for (int32_t i = 0; i < n; ++i) dpos[p.pos[i]] = t.row_ptr[i] + (int32_t)lu.lrow[i].size();
  T_TRY(t_up(t, dpos, &t.dpos, err));
  T_TRY(t_alloc(t, t.n_flat, &t.f, err));
  // G_x and G_x^T by tree rows
  t.nnz_gx = (int32_t)net.gx.nnz();
  for (int tr = 0; tr < 2; ++tr) {
    std::vector<int32_t> ptr(n + 1, 0), col(t.nnz_gx), src(t.nnz_gx);
    auto at = [&](int32_t x) { return p.pos[lu.iperm[x]]; };
    for (int32_t r = 0; r < n; ++r)
      for (int32_t e = net.gx.ptr[r]; e < net.gx.ptr[r + 1]; ++e) ptr[at(tr ? net.gx.col[e] : r) + 1]++;
    for (int32_t i = 0; i < n; ++i) ptr[i + 1] += ptr[i];
    std::vector<int32_t> fill(ptr.begin(), ptr.end() - 1);
    for (int32_t i = 0; i < n; ++i) {  // rows in tree order: ascending tree columns for G_x^T
      const int32_t r = order[i];
      for (int32_t e = net.gx.ptr[r]; e < net.gx.ptr[r + 1]; ++e) {
        const int32_t c = at(net.gx.col[e]);
        const int32_t k = fill[tr ? c : i]++;
        col[k] = tr ? i : c;
        src[k] = e;
      }
    }
    T_TRY(t_up(t, ptr, tr ? &d.at_ptr : &d.an_ptr, err));
    T_TRY(t_up(t, col, tr ? &d.at_col : &d.an_col, err));
    T_TRY(t_up(t, src, tr ? &t.at_src : &t.an_src, err));
    double *v = nullptr;
    T_TRY(t_alloc(t, t.nnz_gx, &v, err));
    (tr ? d.at_val : d.an_val) = v;
  }
  T_TRY(t_alloc(t, t.nnz_gx, &t.gxv, err));
  // arrays filled from the host per operating point
  double *gv = nullptr, *gtv = nullptr;
  T_TRY(t_alloc(t, t.gp_src.size(), &gv, err));
  T_TRY(t_alloc(t, t.gpt_src.size(), &gtv, err));
  d.gp_val = gv;
  d.gpt_val = gtv;
  TreeBus *bus = nullptr;
  TreeInc *inc = nullptr;
  T_TRY(t_alloc(t, net.n_bus, &bus, err));
  T_TRY(t_alloc(t, 2 * (size_t)net.n_br, &inc, err));
  d.bus = bus;
  d.inc = inc;
  int2 *sx = nullptr;
  double2 *sg = nullptr;
  T_TRY(t_alloc(t, net.n_bus, &sx, err));  // at most every bus touches the slack
  T_TRY(t_alloc(t, net.n_bus, &sg, err));
  d.slack_x = sx;
  d.slack_g = sg;
  T_TRY(t_alloc(t, 1, &t.dd, err));
  // a launch's LDS is laid out for the largest node of every network in it,
  // so the kernels' bound is the whole LDS a workgroup may have
  const void *kernels[] = {
      reinterpret_cast<const void *>(&tree_leaf<double, true, false>),
      reinterpret_cast<const void *>(&tree_leaf<double, false, false>),
      reinterpret_cast<const void *>(&tree_upper<double, true, false>),
      reinterpret_cast<const void *>(&tree_upper<double, false, false>),
      reinterpret_cast<const void *>(&tree_top<double, false>),
      reinterpret_cast<const void *>(&tree_leaf<float, true, false>),
      reinterpret_cast<const void *>(&tree_leaf<float, false, false>),
      reinterpret_cast<const void *>(&tree_upper<float, true, false>),
      reinterpret_cast<const void *>(&tree_upper<float, false, false>),
      reinterpret_cast<const void *>(&tree_top<float, false>),
      reinterpret_cast<const void *>(&tree_leaf<double, true, true>),
      reinterpret_cast<const void *>(&tree_upper<double, true, true>),
      reinterpret_cast<const void *>(&tree_top<double, true>),
      reinterpret_cast<const void *>(&tree_invert),
  };
  for (const void *k : kernels) T_TRY(lds_bound(k, kTreeLds, err));
  return RH_OK;
}

// Values of the solved operating point.
rh_status tree_refresh(Network &net, DevTree &t, const double *d_factors, std::string &err) {
  const LuPlan &lu = net.lu;
  const TreePlan &p = t.plan;
  TreeDesc &d = t.d;
  const int32_t n = lu.n;
  const double *f = d_factors;
  if (!f) {
    std::vector<double> flat(t.n_flat);
    for (int32_t i = 0; i < n; ++i) {
      double *r = flat.data() + t.row_ptr[i];
      r = std::copy(lu.lval[i].begin(), lu.lval[i].end(), r);
      std::copy(lu.uval[i].begin(), lu.uval[i].end(), r);
    }
    HIP_TRY(hipMemcpy(t.f, flat.data(), flat.size() * sizeof(double), hipMemcpyHostToDevice));
    f = t.f;
  }
  if (t.n_ents)
    hipLaunchKernelGGL(tree_fill, dim3((t.n_ents + 255) / 256), dim3(256), 0, nullptr, f, t.lo, t.up, t.dg, t.n_ents,
                       t.vl, t.vu);
  double *m[4];
  float *m32[4];
  for (int q = 0; q < 4; ++q) {
    m[q] = const_cast<double *>(d.m64[q]);
    m32[q] = const_cast<float *>(d.m32[q]);
  }
  if (t.n_cols)
    hipLaunchKernelGGL(tree_invert, dim3(t.n_cols, 2), dim3(64), (size_t)p.max_rows * kD * 2 * sizeof(double), nullptr,
                       d.nodes, t.cols, t.ent_ptr, t.col, (const double *)t.vl, (const double *)t.vu, t.map, f,
                       t.dpos, m[0], m[2], m[3], m[1], t.node32, make_int2(d.first32[0], d.first32[1]), m32[0], m32[2],
                       m32[3], m32[1]);
  HIP_TRY(hipGetLastError());
  // G_x, and its norms
  HIP_TRY(hipMemcpy(t.gxv, net.gx.val.data(), (size_t)t.nnz_gx * sizeof(double), hipMemcpyHostToDevice));
  hipLaunchKernelGGL(tree_gather, dim3((t.nnz_gx + 255) / 256), dim3(256), 0, nullptr, (const double *)t.gxv, t.an_src,
                     t.nnz_gx, const_cast<double *>(d.an_val));
  hipLaunchKernelGGL(tree_gather, dim3((t.nnz_gx + 255) / 256), dim3(256), 0, nullptr, (const double *)t.gxv, t.at_src,
                     t.nnz_gx, const_cast<double *>(d.at_val));
  HIP_TRY(hipGetLastError());
  d.norm_n = d.norm_t = 0.0;
  {
    std::vector<double> cs(n, 0.0);
    for (int32_t r = 0; r < n; ++r) {
      double s = 0.0;
      for (int32_t e = net.gx.ptr[r]; e < net.gx.ptr[r + 1]; ++e) {
        const double v = std::fabs(net.gx.val[e]);
        s += v;
        cs[net.gx.col[e]] += v;
      }
      d.norm_n = std::max(d.norm_n, s);
    }
    for (double v : cs) d.norm_t = std::max(d.norm_t, v);
  }
  // G_p
  std::vector<double> gv(t.gp_src.size()), gtv(t.gpt_src.size());
  for (size_t e = 0; e < gv.size(); ++e) gv[e] = net.gp.val[t.gp_src[e]];
  for (size_t e = 0; e < gtv.size(); ++e) gtv[e] = net.gp.val[t.gpt_src[e]];
  if (!gv.empty()) {
    HIP_TRY(hipMemcpy(const_cast<double *>(d.gp_val), gv.data(), gv.size() * 8, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(const_cast<double *>(d.gpt_val), gtv.data(), gtv.size() * 8, hipMemcpyHostToDevice));
  }
  // projection
  auto tx = [&](int32_t b) { return net.th_x[b] >= 0 ? p.pos[lu.iperm[net.th_x[b]]] : -1; };
  auto vs = [&](int32_t b) { return net.v_x[b] >= 0 ? p.pos[lu.iperm[net.v_x[b]]] : -net.v_p[b] - 1; };
  const Tape &tp = net.tape;
  std::vector<TreeBus> bus(net.n_bus);
  std::vector<TreeInc> inc;
  inc.reserve(tp.inc_other.size());
  for (int32_t i = 0; i < net.n_bus; ++i) {
    const int32_t b = t.bus_order[i];
    TreeBus &B = bus[i];
    B = TreeBus{tx(b), vs(b), (int32_t)inc.size(), 0, tp.bus_v[b], tp.bus_sth[b], tp.bus_sv[b], 0.0};
    for (int32_t q = tp.inc_ptr[b]; q < tp.inc_ptr[b + 1]; ++q) {
      const int32_t o = tp.inc_other[q];
      inc.push_back({tp.inc_K[q], tp.inc_Hps[q], tp.inc_H[q], tp.inc_A2[q], tp.inc_vo[q], tx(o), vs(o)});
    }
    B.inc1 = (int32_t)inc.size();
  }
  if (inc.size() > 2 * (size_t)net.n_br) {
    err = "internal: more incidences than branch ends";
    return RH_EDEVICE;
  }
  HIP_TRY(hipMemcpy(const_cast<TreeBus *>(d.bus), bus.data(), bus.size() * sizeof(TreeBus), hipMemcpyHostToDevice));
  if (!inc.empty())
    HIP_TRY(hipMemcpy(const_cast<TreeInc *>(d.inc), inc.data(), inc.size() * sizeof(TreeInc), hipMemcpyHostToDevice));
  d.n_slack = (int32_t)tp.slack_bus.size();
  std::vector<int2> sx(d.n_slack);
  std::vector<double2> sg(d.n_slack);
  for (int32_t q = 0; q < d.n_slack; ++q) {
    sx[q] = make_int2(tx(tp.slack_bus[q]), vs(tp.slack_bus[q]));
    sg[q] = make_double2(tp.slack_gth[q], tp.slack_gv[q]);
  }
  if (d.n_slack > net.n_bus) {
    err = "internal: more slack terms than buses";
    return RH_EDEVICE;
  }
  if (d.n_slack) {
    HIP_TRY(hipMemcpy(const_cast<int2 *>(d.slack_x), sx.data(), sx.size() * sizeof(int2), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(const_cast<double2 *>(d.slack_g), sg.data(), sg.size() * sizeof(double2), hipMemcpyHostToDevice));
  }
  HIP_TRY(hipMemcpy(t.dd, &d, sizeof d, hipMemcpyHostToDevice));
  return RH_OK;
}

}  // namespace

rh_status tree_upload(Network &net, const double *d_factors, bool *used, std::string &err) {
  *used = false;
  if (!net.dtree) {
    DevTree *t = new DevTree();
    net.dtree = t;
    t->device = net.ctx->device;
    rh_status s;
    try {
      s = tree_build(net, *t, err);
    } catch (...) {
      device_tree_free(net);
      throw;
    }
    if (s != RH_OK) {
      device_tree_free(net);
      return s;
    }
  }
  if (!net.dtree->plan.ok) return RH_OK;
  rh_status s = tree_refresh(net, *net.dtree, d_factors, err);
  *used = s == RH_OK;
  return s;
}

void tree_steps(const DevTree *t, int32_t &fwd, int32_t &bwd) { fwd = bwd = t->d.n_tiers; }

void device_tree_free(Network &net) {
  DevTree *t = net.dtree;
  if (!t) return;
  (void)hipSetDevice(t->device);
  (void)hipDeviceSynchronize();
  for (void *p : t->allocs) (void)hipFree(p);
  delete t;
  net.dtree = nullptr;
}

int64_t tree_bytes(const DevTree *t) { return t ? t->bytes : 0; }

// A round's scratch and chunks at most.  A round costs its launches' chains
// (13 of 5 to 25 us at 10k buses) besides its traffic, so the fewer the better,
// even though its vectors then leave the caches: the full Hessian at 10k
// buses (175 chunks of 6 MB) takes 4.39 ms in rounds of 8, 2.04 in rounds of
// 32, 1.75 in rounds of 64 and 1.59 in one; four batches of 128 at 70k (32
// chunks of 50 MB) 4.17 ms in rounds of 256 MB, 2.93 of 1 GB, 2.61 in one.
constexpr size_t kRoundBytes = size_t(2) << 30;
constexpr int32_t kRoundChunks = 256;

size_t TreeWork::bytes() const { return (size_t)(data + (int64_t)round * norm_doubles()) * sizeof(double); }
int64_t TreeWork::norm_doubles() const { return (int64_t)norm_iters * 4 * kD; }

TreeWork tree_work(const std::vector<TreeRequest> &req, int32_t refine, size_t most) {
  TreeWork w;
  w.norm_iters = refine >= 0 ? refine + 1 : 0;
  for (const TreeRequest &r : req) w.chunks += (r.k + kD - 1) / kD;
  const int64_t room = (int64_t)(std::min(most, kRoundBytes) / sizeof(double));
  // the requests' chunks in rounds of at most `per`, a request split where a
  // round ends; the number of rounds
  auto fill = [&](int32_t per) {
    w.items.clear();
    w.round = 0;
    w.data = 0;
    int32_t used = 0, round = 0;
    int64_t data = 0;
    for (const TreeRequest &r : req) {
      const TreeDesc &d = r.t->d;
      // FP64: Z, Y, the update rows, W and Y_p; refined: FP64 residual and
      // solution, the FP32 correction and its update rows
      const int64_t u = refine >= 0 ? ((int64_t)d.n_x + d.n_u + 1) / 2 : d.n_u;
      const int64_t rows = 2 * (int64_t)d.n_x + u + 2 * (int64_t)d.n_p,
                    size = (rows * kD + kTreeLine - 1) / kTreeLine * kTreeLine;
      bool open = false;  // the last item is this request's, of this round
      for (int32_t d0 = 0; d0 < r.k; d0 += kD) {
        if (used == per || (used > 0 && std::max(w.data, data + size) + std::max(w.round, used + 1) * w.norm_doubles() > room)) {
          ++round;
          used = 0;
          data = 0;
          open = false;
        }
        if (!open) {
          TreeItem it{};
          it.td = r.t->dd;
          it.W = r.W ? r.W + (int64_t)d0 * r.ldw : nullptr;
          it.HW = r.HW + (int64_t)d0 * r.ldhw;
          it.ldw = r.ldw;
          it.ldhw = r.ldhw;
          it.identity_from = r.identity_from < 0 ? -1 : r.identity_from + d0;
          it.chunk0 = used;
          it.round = round;
          it.at = (int32_t)((data - used * size) / kTreeLine);
          it.stride = (int32_t)(size / kTreeLine);
          it.rinfo = r.rinfo ? r.rinfo + 4 * (int64_t)d0 : nullptr;
          w.items.push_back(it);
          open = true;
        }
        w.items.back().k += std::min(kD, r.k - d0);
        w.items.back().chunks += 1;
        data += size;
        ++used;
        w.data = std::max(w.data, data);
        w.round = std::max(w.round, used);
      }
    }
    return round + 1;
  };
  // as many rounds as that takes, of equal length
  const int32_t rounds = fill(kRoundChunks);
  if (rounds > 1) fill((w.chunks + rounds - 1) / rounds);
  return w;
}

rh_status tree_launch(const std::vector<TreeRequest> &req, const TreeWork &work, const TreeItem *items, double *scratch,
                      int32_t refine, double tol, long long *stamps, hipStream_t s, std::string &err) {
  if (work.chunks <= 0) return RH_OK;
  const std::vector<TreeItem> &host_items = work.items;
  // the largest of every network's dimensions shapes the launches
  std::vector<int32_t> nodes(kTreeTiers, 0);
  int32_t tiers = 0, n_p = 0, n_x = 0, n_bus = 0, n_gp = 0, leaf = 0, upper = 0, top = 0;
  bool dirs = false;
  for (const TreeRequest &r : req) {
    const TreePlan &p = r.t->plan;
    const TreeDesc &d = r.t->d;
    const int32_t low = d.n_tiers - 1;  // tiers below the top
    for (int32_t q = 0; q < low; ++q) {
      nodes[q] = std::max(nodes[q], p.tier[q + 1] - p.tier[q]);
      (q == 0 ? leaf : upper) = std::max(q == 0 ? leaf : upper, p.max_tiles[q]);
    }
    tiers = std::max(tiers, low);
    top = std::max(top, p.max_tiles[low]);
    n_p = std::max(n_p, d.n_p);
    n_x = std::max(n_x, d.n_x);
    n_bus = std::max(n_bus, d.n_bus);
    n_gp = std::max(n_gp, d.n_gp_rows);
    dirs = dirs || r.identity_from < 0;
  }
  const bool ref = refine >= 0;
  const size_t el = ref ? sizeof(float) : sizeof(double), row = kT * kD * el;  // a row tile of one chunk
  const size_t parts = kUpperWaves * kTileVals * el;  // sums that span waves
  const size_t top_lds = 2 * (size_t)top * row + parts;
  if (std::max({2 * leaf * kT * kD * sizeof(double), upper * row + parts, top_lds}) > kTreeLds) {
    err = "internal: node larger than the LDS";
    return RH_EDEVICE;
  }
  TreeArgs a{};
  a.tol = tol;
  a.scratch = scratch;
  a.norm_iters = work.norm_iters;
  a.norms = ref ? scratch + work.data : nullptr;
  a.stamps = stamps;
  for (size_t i0 = 0, i1; i0 < host_items.size(); i0 = i1) {
    uint32_t nc = 0;
    for (i1 = i0; i1 < host_items.size() && host_items[i1].round == host_items[i0].round; ++i1)
      nc = (uint32_t)(host_items[i1].chunk0 + host_items[i1].chunks);
    a.n_items = (int32_t)(i1 - i0);
    a.n_chunks = (int32_t)nc;
    a.items = a.n_items > 1 ? items + i0 : nullptr;
    a.one = host_items[i0];
    auto tier_launch = [&](int32_t q, bool fwd, int which, int iter) {
      // node x lands on the same XCD for every chunk when the row of the
      // grid is a multiple of eight: its matrices stay in that XCD's L2
      const uint32_t gx = q == 0 ? (uint32_t)((nodes[0] + 7) & ~7) : (uint32_t)nodes[q];
      const uint32_t most = q == 0 ? std::max<uint32_t>(1, kLeafGroups / gx) : nc;
      const int per = std::min<int>(kChunkRun, (int)((nc + most - 1) / most));
      const dim3 grid(gx, (nc + per - 1) / per), block((q == 0 ? kLeafWaves : kUpperWaves) * 64);
      a.lds_rows = (q == 0 ? leaf : upper) * kT;
      const size_t lds = q == 0 ? (per > 1 ? 2 : 1) * (size_t)a.lds_rows * kD * sizeof(double)
                                : (size_t)a.lds_rows * kD * el + parts;
      const bool sp = fwd && !ref && which == 0;
      if (q == 0) {
#define TREE_LEAF(T, F, S) hipLaunchKernelGGL((tree_leaf<T, F, S>), grid, block, lds, s, a, which, iter, per)
        if (ref && fwd)
          TREE_LEAF(float, true, false);
        else if (ref)
          TREE_LEAF(float, false, false);
        else if (sp)
          TREE_LEAF(double, true, true);
        else if (fwd)
          TREE_LEAF(double, true, false);
        else
          TREE_LEAF(double, false, false);
#undef TREE_LEAF
      } else {
#define TREE_UPPER(T, F, S) hipLaunchKernelGGL((tree_upper<T, F, S>), grid, block, lds, s, a, q, which, iter)
        if (ref && fwd)
          TREE_UPPER(float, true, false);
        else if (ref)
          TREE_UPPER(float, false, false);
        else if (sp)
          TREE_UPPER(double, true, true);
        else if (fwd)
          TREE_UPPER(double, true, false);
        else
          TREE_UPPER(double, false, false);
#undef TREE_UPPER
      }
    };
    auto solve = [&](int which, int iter) {
      for (int32_t q = 0; q < tiers; ++q) tier_launch(q, true, which, iter);
      const dim3 tb(kUpperWaves * 64);
      if (ref)
        hipLaunchKernelGGL((tree_top<float, false>), dim3(nc), tb, top_lds, s, a, which, iter);
      else if (which == 0)
        hipLaunchKernelGGL((tree_top<double, true>), dim3(nc), tb, top_lds, s, a, which, iter);
      else
        hipLaunchKernelGGL((tree_top<double, false>), dim3(nc), tb, top_lds, s, a, which, iter);
      for (int32_t q = tiers - 1; q >= 0; --q) tier_launch(q, false, which, iter);
      if (ref) {
        const uint32_t gx = (uint32_t)((n_x + kResRows - 1) / kResRows), most = std::max<uint32_t>(1, kResGroups / gx);
        const int per = std::min<int>(kChunkRun, (int)((nc + most - 1) / most));
        hipLaunchKernelGGL(tree_residual, dim3(gx, (nc + per - 1) / per), dim3(512), 0, s, a, which, iter, per);
      }
    };
    if (dirs || ref || stamps)
      hipLaunchKernelGGL(tree_in, dim3((n_p + kMoveRows - 1) / kMoveRows, nc), dim3(256), 0, s, a);
    if (ref) hipLaunchKernelGGL(tree_spmul, dim3((n_gp + 15) / 16, nc), dim3(256), 0, s, a);
    for (int it = 0; it <= std::max(0, refine); ++it) solve(0, it);
    const uint32_t px = ((n_bus + kProjBuses - 1) / kProjBuses + 7) & ~7;
    const uint32_t pmost = std::max<uint32_t>(1, kProjGroups / px);
    const int pper = (int)((nc + pmost - 1) / pmost);
    hipLaunchKernelGGL(tree_project, dim3(px, (nc + pper - 1) / pper), dim3(256), 0, s, a, pper);
    for (int it = 0; it <= std::max(0, refine); ++it) solve(1, it);
    hipLaunchKernelGGL(tree_out, dim3((n_p + kMoveRows - 1) / kMoveRows, nc), dim3(256), 0, s, a);
    HIP_TRY(hipGetLastError());
  }
  return RH_OK;
}

}  // namespace rh
