// Dense FP64 Cholesky factorisation and solves on the device: the dense
// linear system H_t d_t = -g_t of the real-time tracking update (Sec. 6.3,
// eq. (qp_rto)), whose matrix is the reduced Hessian that stays resident in
// HBM after Algorithm 2.
//
// A is column-major, n x n, leading dimension lda; only its lower triangle
// (diagonal included) is read and it is overwritten by L with A = L L^T.
// Right-looking, in panels of kNB columns, one launch per panel.  Its first
// workgroups finish the panel, a strip each: the kNB rows of the diagonal
// block (every workgroup again) and kNB rows below it.  They take the update
// of the panel before (FP64 MFMA, 16 x 16 x 4), then the factorisation in
// sub-panels of 16 columns in LDS: the diagonal tile by one wave in registers,
// the rows below it by substitution, a row per thread, the rest of the strip
// by MFMA.  The other workgroups take the update of the panel before on the
// columns right of the panel, in 64 x 64 tiles: a lookahead of one panel.
// A failed pivot (not positive, or not finite) stores its column + 1 in a
// status word, which the first panel sets; every later kernel reads it first
// and does nothing.
// The forward sweep L Y = B rides along: the right-hand sides are extra rows
// of the augmented matrix [A; B^T], so that at the end B holds Y.
// chol_back_block then solves L^T X = Y a block of 64 unknowns per launch,
// from the last.
//
// What bounds it: a panel's launch is a chain of two trips to memory, the
// update (7 us) and four sub-panels (16 pivots and a substitution of 16 each,
// 4.5 us), about 26 us, or the update's traffic (a 64 x 64 tile moves 128 KB
// for 0.5 MFLOP: 63 us at 4,555 columns) where the trailing matrix is large.
// Panels of 32 columns, with the update of the next panel's columns in a
// launch of its own, took 20 us for half the columns, and the solves L^T X = Y
// 17 us a block where they take 7 now; 4,555 columns with one right-hand
// side: 5.3 ms before, 3.4 ms now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "rh_internal.h"

namespace rh {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kNB = 64;  // panel width, rows of a strip below the diagonal block, trailing-update tile
constexpr int kSub = 16;  // columns of a sub-panel
constexpr int kThreads = 512;  // of a panel's launch

__device__ __forceinline__ double rdlane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// 1 / sqrt(d) for a pivot d: the hardware reciprocal square root (to 2^-23)
// refined by one step of third order on f(r) = 1 / r^2 - d,
// r (1 + e / 2 + 3 e^2 / 8) with e = 1 - d r^2, whose error is of the order
// of e^3 < 2^-65: a shorter dependency chain than a square root and a
// division, or than two Newton-Raphson steps.  Pivots below 2^-900 are scaled
// by 2^1000 (exactly, a power of two) and the result by 2^500, so that the
// estimate never sees a denormal; a branch, as all lanes have the same pivot.
__device__ __forceinline__ double pivot_rsqrt(double d) {
  auto refined = [](double x) {
    const double r = __builtin_amdgcn_rsq(x), e = fma(-x * r, r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
  };
  double r = refined(d);
  if (__builtin_expect(d < 0x1p-900, 0)) r = refined(d * 0x1p+1000) * 0x1p+500;
  return r;
}

// Lane C of each group of 16 lanes to all its lanes.
template <int C>
__device__ __forceinline__ double group_bcast(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + C, 0xF, 0xF, true);
}
// Step C of L L^T of a 16 x 16 tile: lane r of each group of 16 lanes holds
// row r (by symmetry also column r), register c its entry c, and ends with
// its row of L (entries right of the diagonal are of no use).  The groups do
// the same, so that every broadcast stays within one.  rinv: 1 / sqrt of the
// pivots; bad: the first pivot that is not positive and finite.  The empty asm
// statements materialise d[k] at the end of the step: the compiler would
// otherwise sink each entry's updates down to its own step, where they are a
// serial chain.  A tile takes 1.2 us.
template <int K, int C>
__device__ __forceinline__ void chol_row(double (&d)[kSub], double l) {
  if constexpr (K < kSub) {
    d[K] = fma(-group_bcast<K>(l), l, d[K]);  // (by symmetry entry K of row r loses L(K, C) L(r, C))
    chol_row<K + 1, C>(d, l);
  }
}
template <int C>
__device__ __forceinline__ void chol_tile(double (&d)[kSub], double (&rinv)[kSub], int32_t &bad) {
  if constexpr (C < kSub) {
    const double dcc = group_bcast<C>(d[C]);
    if (bad < 0 && !(dcc > 0.0 && dcc <= 1.7976931348623157e308)) bad = C;
    // column C scaled by 1 / sqrt(d_CC); on the diagonal this gives the pivot
    // d_CC / sqrt(d_CC) itself (within an ulp of sqrt(d_CC))
    rinv[C] = pivot_rsqrt(dcc);
    d[C] *= rinv[C];
    chol_row<C + 1, C>(d, d[C]);
#pragma unroll
    for (int k = C + 1; k < kSub; ++k) asm volatile("" : "+v"(d[k]));
    chol_tile<C + 1>(d, rinv, bad);
  }
}

// F = A (lower triangle) with tau added on the diagonal; columns per block.
__global__ __launch_bounds__(256) void dense_shift_copy(const double *A, int64_t lda, double *F, int64_t ldf,
                                                        int32_t n, double tau) {
  const int32_t j = blockIdx.x;
  for (int32_t i = j + threadIdx.x; i < n; i += 256) {
    const double v = A[i + (int64_t)j * lda];
    F[i + (int64_t)j * ldf] = i == j ? v + tau : v;
  }
}

__global__ __launch_bounds__(256) void dense_diag(const double *A, int64_t lda, int32_t n, double *out) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = A[i + (int64_t)i * lda];
}

__global__ __launch_bounds__(256) void dense_neg(const double *a, double *b, int32_t n) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = -a[i];
}

// The augmented matrix [A; B^T]: entry c of row r is at row(r).p[c * row(r).ld].
struct Aug {
  double *A, *B;
  int64_t lda, ldb;
  int32_t n, rows;  // rows: n and the right-hand sides
};
struct AugRow {
  double *p;
  int64_t ld;
};
__device__ __forceinline__ AugRow aug_row(const Aug &M, int32_t r) {
  return r < M.n ? AugRow{M.A + r, M.lda} : AugRow{M.B + (int64_t)(r - M.n) * M.ldb, 1};
}

// The MFMA forms D = S_k S_i^T from 16 x 4 slabs of a panel, S_k over columns
// and S_i over rows of the matrix, so that D[a][b] belongs to row b, column
// a: a lane's four outputs then lie along one row and 16 lanes hold 16
// consecutive rows.  Operand layout of v_mfma_f64_16x16x4f64 (measured on
// gfx950): lane l holds A-operand (l % 16, l / 16) and B-operand (l / 16,
// l % 16); output register q of lane l is D[4 q + l / 16][l % 16].
//
// acc -= (panel j's rows r0 ..) (panel j's rows c0 ..)^T, RI x CK tiles of a
// wave; entries of rows past `rows` (columns past n) are zero.
template <int RI, int CK>
__device__ __forceinline__ void panel_product(const Aug &M, int32_t j, int32_t r0, int32_t c0, int lane,
                                              v4d (&acc)[CK][RI]) {
  const int l16 = lane & 15, g = lane >> 4;
  const double *pr[RI], *pc[CK];
  int64_t sr[RI], sc[CK];
  bool okr[RI], okc[CK];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int32_t r = r0 + 16 * i + l16;
    okr[i] = r < M.rows;
    const AugRow a = aug_row(M, okr[i] ? r : j);
    pr[i] = a.p + (int64_t)(j + g) * a.ld;
    sr[i] = 4 * a.ld;
  }
#pragma unroll
  for (int k = 0; k < CK; ++k) {
    const int32_t c = c0 + 16 * k + l16;
    okc[k] = c < M.n;
    pc[k] = M.A + (okc[k] ? c : j) + (int64_t)(j + g) * M.lda;
    sc[k] = 4 * M.lda;
  }
  // groups of two steps: the next group's operands are loaded meanwhile
  constexpr int kG = 2;
  double xr[2][kG][RI], xc[2][kG][CK];
  auto load = [&](int s, double (&vr)[kG][RI], double (&vc)[kG][CK]) {
#pragma unroll
    for (int h = 0; h < kG; ++h) {
#pragma unroll
      for (int i = 0; i < RI; ++i) vr[h][i] = pr[i][(s + h) * sr[i]];
#pragma unroll
      for (int k = 0; k < CK; ++k) vc[h][k] = pc[k][(s + h) * sc[k]];
    }
  };
  load(0, xr[0], xc[0]);
#pragma unroll
  for (int s = 0; s < kNB / 4; s += kG) {
    const int b = (s / kG) & 1;
    if (s + kG < kNB / 4) load(s + kG, xr[b ^ 1], xc[b ^ 1]);
#pragma unroll
    for (int h = 0; h < kG; ++h)
#pragma unroll
      for (int k = 0; k < CK; ++k)
#pragma unroll
        for (int i = 0; i < RI; ++i)
          acc[k][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(okc[k] ? -xc[b][h][k] : 0.0, okr[i] ? xr[b][h][i] : 0.0,
                                                           acc[k][i], 0, 0, 0);
  }
}

constexpr int kStrip = 2 * kNB;      // rows of a strip: the diagonal block's, and as many below
constexpr int kStripLd = kStrip + 4;  // (columns of the strip start at other banks)
struct PanelLds {
  double S[kNB * kStripLd];  // the strip, column by column
  __align__(16) double D[kSub * kSub];
  __align__(16) double rinv[kSub];
  int32_t bad;
};

// Strip blk of panel j.
// The diagonal block's factor goes to `diag` where there are other strips,
// which may still be reading the block.
__device__ __forceinline__ void panel_strip(const Aug &M, int32_t j, int32_t blk, int32_t strips, int32_t *info, double *diag,
                                            PanelLds &L) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g = lane >> 4;
  const int32_t nb = min(kNB, M.n - j), below = j + nb + blk * kNB;  // first row below
  __builtin_amdgcn_s_setprio(3);  // the chain, ahead of the tiles' waves on the same SIMD
  // row i of the strip; rows (and columns) past nb of the diagonal block are
  // completed by the identity
  auto row_of = [&](int i) { return i < kNB ? (i < nb ? j + i : M.rows) : below + i - kNB; };
  {
    // a wave's 16 rows, with the update of the panel before
    const int i = wave * 16 + l16;
    const int32_t r = row_of(i);
    const AugRow a = aug_row(M, r < M.rows ? r : j);
    double cur[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 16 * k + 4 * q + g;
        // of the diagonal block the lower triangle, mirrored
        const double *p = i < kNB && c > i ? M.A + (j + c) + (int64_t)(j + i) * M.lda : a.p + (int64_t)(j + c) * a.ld;
        cur[k][q] = 0.0;
        if (r < M.rows && c < nb) cur[k][q] = *p;
      }
    v4d acc[4][1];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k][0] = v4d{0.0, 0.0, 0.0, 0.0};
    // (rows 0 .. 63 and 64 .. of the strip are consecutive rows each)
    if (j > 0) panel_product<1, 4>(M, j - kNB, wave * 16 < kNB ? j + wave * 16 : below + wave * 16 - kNB, j, lane, acc);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 16 * k + 4 * q + g;
        // (the product reaches past nb: those rows and columns stay the identity)
        L.S[c * kStripLd + i] = r < M.rows && c < nb ? cur[k][q] + acc[k][0][q] : i == c ? 1.0 : 0.0;
      }
  }
  if (tid == 0) L.bad = -1;
  __syncthreads();
  auto factor = [&](int s) {  // diagonal tile s (one wave)
    double d[kSub], rinv[kSub];
    int32_t bad = -1;
    double *T = &L.S[s * kSub * kStripLd + s * kSub];
    // entry c of row l16 from the lower triangle
#pragma unroll
    for (int c = 0; c < kSub; ++c) d[c] = T[min(c, l16) * kStripLd + max(c, l16)];
    chol_tile<0>(d, rinv, bad);
    if (bad >= 0 && lane == 0 && L.bad < 0) L.bad = s * kSub + bad;
    if (g == 0) {
#pragma unroll
      for (int c = 0; c < kSub; ++c) {
        L.D[c * kSub + l16] = d[c];  // column by column
        T[c * kStripLd + l16] = d[c];
        if (l16 == c) L.rinv[c] = rinv[c];
      }
    }
  };
  if (wave == 0) factor(0);
  // (sub-panels past nb are the identity)
  for (int s = 0; s * kSub < nb; ++s) {
    __syncthreads();
    if (L.bad >= 0) break;
    const int first = (s + 1) * kSub;  // first row below the tile
    if (first + tid < kStrip) {
      double v[kSub];
      double *P = &L.S[s * kSub * kStripLd + first + tid];
#pragma unroll
      for (int c = 0; c < kSub; ++c) v[c] = P[c * kStripLd];
      // column c of the tile is read a step ahead
      double l[2][kSub];
      const double2 *Dc = reinterpret_cast<const double2 *>(L.D), *rv = reinterpret_cast<const double2 *>(L.rinv);
      double ri[kSub];
#pragma unroll
      for (int m = 0; m < kSub / 2; ++m) {
        const double2 x = Dc[m], y = rv[m];
        l[0][2 * m] = x.x;
        l[0][2 * m + 1] = x.y;
        ri[2 * m] = y.x;
        ri[2 * m + 1] = y.y;
      }
#pragma unroll
      for (int c = 0; c < kSub; ++c) {
        if (c + 1 < kSub) {
#pragma unroll
          for (int m = (c + 2) / 2; m < kSub / 2; ++m) {
            const double2 x = Dc[(c + 1) * (kSub / 2) + m];
            l[(c + 1) & 1][2 * m] = x.x;
            l[(c + 1) & 1][2 * m + 1] = x.y;
          }
        }
        v[c] *= ri[c];
#pragma unroll
        for (int m = c + 1; m < kSub; ++m) v[m] = fma(-v[c], l[c & 1][m], v[m]);
      }
#pragma unroll
      for (int c = 0; c < kSub; ++c) P[c * kStripLd] = v[c];
    }
    __syncthreads();
    // the strip right of the sub-panel: tile column k, tile row i >= k; the
    // first wave takes the next diagonal tile and factors it
    int t = 0;
    for (int k = s + 1; k < kNB / kSub; ++k)
      for (int i = k; i < kStrip / kSub; ++i, ++t) {
        const bool next = k == s + 1 && i == k;
        if (next ? wave != 0 : wave != 1 + (t - 1) % (kThreads / 64 - 1)) continue;
        v4d acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = L.S[(k * kSub + 4 * q + g) * kStripLd + i * kSub + l16];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const double *c = &L.S[(s * kSub + 4 * h + g) * kStripLd + l16];
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-c[k * kSub], c[i * kSub], acc, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) L.S[(k * kSub + 4 * q + g) * kStripLd + i * kSub + l16] = acc[q];
        if (next) {
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          factor(s + 1);
        }
      }
  }
  __syncthreads();
  if (blk == 0 && tid == 0 && (L.bad >= 0 || j == 0)) *info = L.bad >= 0 ? j + L.bad + 1 : 0;
  if (L.bad >= 0) return;
  const int i = tid & (kStrip - 1);
  const int32_t r = row_of(i);
  if (i < kNB) {
    if (strips == 1) {  // (nothing else reads the block)
      for (int c = tid / kStrip; c <= i && i < nb; c += kThreads / kStrip)
        M.A[r + (int64_t)(j + c) * M.lda] = L.S[c * kStripLd + i];
    } else if (blk == 0)
      for (int c = tid / kStrip; c < kNB; c += kThreads / kStrip) diag[c * kNB + i] = L.S[c * kStripLd + i];
  } else if (r < M.rows) {
    const AugRow a = aug_row(M, r);
    for (int c = tid / kStrip; c < nb; c += kThreads / kStrip) a.p[(int64_t)(j + c) * a.ld] = L.S[c * kStripLd + i];
  }
}

// Panel j's diagonal block from `diag` into the matrix (lower triangle).
__device__ __forceinline__ void put_diag(const Aug &M, int32_t j, const double *diag) {
  const int32_t nb = min(kNB, M.n - j);
  for (int e = threadIdx.x; e < kNB * kNB; e += blockDim.x) {
    const int i = e % kNB, c = e / kNB;
    if (i < nb && c <= i) M.A[(j + i) + (int64_t)(j + c) * M.lda] = diag[e];
  }
}
// Tile (ti, tk), ti >= tk, of a trailing matrix of T tile columns (and more
// tile rows where there are many right-hand sides) from a linear index.
__device__ __forceinline__ void tri_tile(int32_t b, int32_t T, int32_t &ti, int32_t &tk) {
  const int64_t tri = (int64_t)T * (T + 1) / 2;
  if (b >= tri) {
    ti = T + (int32_t)((b - tri) / T);
    tk = (int32_t)((b - tri) % T);
    return;
  }
  int32_t t = (int32_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while ((int64_t)(t + 1) * (t + 2) / 2 <= b) ++t;
  while ((int64_t)t * (t + 1) / 2 > b) --t;
  ti = t;
  tk = b - (int32_t)((int64_t)t * (t + 1) / 2);
}

// The update of panel j on the 64 x 64 tile (ti, tk) of the matrix from row
// and column j1 on: a 32 x 32 quadrant each for four waves.
__device__ __forceinline__ void update_tile(const Aug &M, int32_t j, int32_t j1, int32_t ti, int32_t tk) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qi = wave >> 1 & 1, qk = wave & 1;
  if (ti == tk && qk > qi) return;  // above the diagonal
  const int32_t r0 = j1 + ti * kNB + qi * 32, c0 = j1 + tk * kNB + qk * 32;
  if (r0 >= M.rows || c0 >= M.n) return;
  const int l16 = lane & 15, g = lane >> 4;
  // (the product is summed up by itself: an entry is rounded to its own size
  // once per panel)
  v4d acc[2][2];
  double cur[2][2][4];
  double *p[2];
  int64_t ld[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int32_t row = r0 + 16 * h + l16;
    const AugRow a = aug_row(M, row < M.rows ? row : j);
    p[h] = a.p;
    ld[h] = a.ld;
  }
  auto in = [&](int h, int k, int q) {
    const int32_t row = r0 + 16 * h + l16, col = c0 + 16 * k + 4 * q + g;
    return row < M.rows && col < M.n && row >= col;
  };
  auto at = [&](int h, int k, int q) { return p[h] + (int64_t)(c0 + 16 * k + 4 * q + g) * ld[h]; };
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        cur[k][h][q] = acc[k][h][q] = 0.0;
        if (in(h, k, q)) cur[k][h][q] = *at(h, k, q);
      }
  panel_product<2, 2>(M, j, r0, c0, lane, acc);
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (in(h, k, q)) *at(h, k, q) = cur[k][h][q] + acc[k][h][q];
}

// Panel j in the first `strips` workgroups; after the first panel also the
// rest of the update of the panel before (T tile columns) in the others,
// which touch none of panel j's columns, and, in the last, that panel's
// diagonal block into its place.  diag: two blocks, taken in turn.
__global__ __launch_bounds__(kThreads, 2) void chol_panel(Aug M, int32_t j, int32_t strips, int32_t T,
                                                         int32_t tiles, int32_t *info, double *diag) {
  __shared__ PanelLds L;
  if (j > 0 && *info) return;  // (the first panel sets the word)
  double *mine = diag + (j / kNB & 1) * kNB * kNB, *before = diag + ((j / kNB & 1) ^ 1) * kNB * kNB;
  const int32_t strips_before = (M.rows - j + kNB - 1) / kNB;  // of the panel before
  if ((int32_t)blockIdx.x < strips) {
    panel_strip(M, j, blockIdx.x, strips, info, mine, L);
  } else if (blockIdx.x + 1 == gridDim.x) {
    if (strips_before > 1) put_diag(M, j - kNB, before);
  } else {
    int32_t ti, tk;
    // two tiles, four waves each
    const int32_t b = 2 * ((int32_t)blockIdx.x - strips) + (threadIdx.x >> 8);
    if (b >= tiles) return;
    tri_tile(b, T, ti, tk);
    update_tile(M, j - kNB, j + kNB, ti, tk);
  }
}

// L^T x = y, one launch per block of 64 unknowns from the last (the rows of
// B above the block already hold z = y - contributions of the later
// blocks).  Every workgroup solves the block's triangle (staged in LDS,
// wave 0) and then updates its 64 rows above, right-looking:
// z_r -= sum_c L(j0 + c, r) x_c, whose 64 entries are contiguous in column r:
// 16 lanes take a column together, loaded before the triangle is solved.
// Workgroup 0 stores the block's x in X (not in B, whose block rows the
// other workgroups may still be reading).  Columns of B: grid y.  diag: the
// block's triangle where it is not in the matrix yet (the last panel's, with
// several strips), or null; the first workgroup then brings it there.
__global__ __launch_bounds__(256) void chol_back_block(double *A, int64_t lda, int32_t n, double *B, int64_t ldb, double *X,
                                                       int32_t j0, const int32_t *info, const double *diag) {
  if (*info) return;
  __shared__ double s_L[64][65];
  __shared__ double s_x[64];
  double *z = B + (int64_t)blockIdx.y * ldb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  const int32_t bs = min(64, n - j0);
  const double *T = diag ? diag : A + j0 + (int64_t)j0 * lda;
  const int64_t ldt = diag ? kNB : lda;
  for (int t = threadIdx.x; t < 64 * 64; t += 256) {
    const int i = t & 63, c = t >> 6;  // consecutive threads: consecutive rows of a column
    s_L[i][c] = (i < bs && c <= i) ? T[i + c * ldt] : 0.0;
  }
  if (diag && blockIdx.x == 0 && blockIdx.y == 0)
    for (int t = threadIdx.x; t < 64 * 64; t += 256) {
      const int i = t & 63, c = t >> 6;
      if (i < bs && c <= i) A[(j0 + i) + (int64_t)(j0 + c) * lda] = diag[t];
    }
  // the group's rows r (columns of L): entries l16 + 16 m of column r
  double v[4][4];
  const int32_t r0 = (int32_t)blockIdx.x * 64 + wave * 16 + g;
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int32_t r = r0 + 4 * h, c = l16 + 16 * m;
      v[h][m] = r < j0 && c < bs ? A[j0 + c + (int64_t)r * lda] : 0.0;
    }
  __syncthreads();
  if (wave == 0) {
    // lane i: z_i and column i of the strictly lower triangle; right-looking
    // from the last unknown: x_c = z_c / L(c, c) (broadcast), then
    // z_i -= L(c, i) x_c on every lane.  Lane i's z stops changing once c
    // passes i (L(c, i) = 0 for c < i here, and its own step comes last), so
    // x_i = z_i / L(i, i) at the end.
    double col[64];
#pragma unroll
    for (int c = 0; c < 64; ++c) col[c] = lane < c ? s_L[c][lane] : 0.0;
    const double rinv = lane < bs ? 1.0 / s_L[lane][lane] : 0.0;
    double zv = lane < bs ? z[j0 + lane] : 0.0;
#pragma unroll
    for (int c = 63; c >= 0; --c) zv = fma(-col[c], rdlane(zv * rinv, c), zv);
    const double xv = zv * rinv;
    s_x[lane] = xv;
    if (blockIdx.x == 0 && lane < bs) X[(int64_t)blockIdx.y * n + j0 + lane] = xv;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) acc = fma(v[h][m], s_x[l16 + 16 * m], acc);
    for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    const int32_t r = r0 + 4 * h;
    if (l16 == 0 && r < j0) z[r] -= acc;
  }
}

__global__ __launch_bounds__(256) void dense_copy_cols(const double *X, int32_t n, double *B, int64_t ldb,
                                                       int32_t nrhs) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nrhs) return;
  const int32_t q = (int32_t)(t / n), i = (int32_t)(t % n);
  B[i + (int64_t)q * ldb] = X[t];
}

}  // namespace

// ---- host side --------------------------------------------------------------

#define DENSE_TRY(expr)                                   \
  do {                                                    \
    hipError_t e_ = (expr);                               \
    if (e_ != hipSuccess) {                               \
      err = std::string(#expr) + ": " + hipGetErrorString(e_); \
      return RH_EDEVICE;                                  \
    }                                                     \
  } while (0)

// The status word's memory: the word (padded) and two diagonal blocks.
constexpr size_t kInfoWords = 32;
size_t dense_info_bytes() { return (kInfoWords + 2 * kNB * kNB) * sizeof(double); }
namespace {
// Panel j's diagonal block there.
const double *diag_of(const int32_t *dinfo, int32_t j) {
  return reinterpret_cast<const double *>(dinfo) + kInfoWords + (j / kNB & 1) * kNB * kNB;
}
}  // namespace

rh_status dense_cholesky(int32_t n, double *A, int64_t lda, double *B, int64_t ldb, int32_t nrhs, int32_t *dinfo,
                         void *stream, std::string &err) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!B) nrhs = 0;
  const Aug M{A, B, lda, ldb, n, n + nrhs};
  double *diag = reinterpret_cast<double *>(dinfo) + kInfoWords;
  for (int32_t j = 0; j < n; j += kNB) {
    const int32_t below = M.rows - j - std::min(kNB, n - j);  // rows under the diagonal block
    const int32_t strips = std::max(1, (below + kNB - 1) / kNB);
    const int64_t T = j > 0 ? std::max(0, (n - j - kNB + kNB - 1) / kNB) : 0;  // tile columns right of the panel
    const int64_t R = T > 0 ? (M.rows - j - kNB + kNB - 1) / kNB : 0;          // tile rows
    const int64_t tiles = T * (T + 1) / 2 + (R - T) * T;
    hipLaunchKernelGGL(chol_panel, dim3((uint32_t)(strips + (tiles + 1) / 2 + (j > 0 ? 1 : 0))), dim3(kThreads), 0, st,
                       M, j, strips, (int32_t)T, (int32_t)tiles, dinfo, diag);
  }
  DENSE_TRY(hipGetLastError());
  return RH_OK;
}

rh_status dense_back_solve(int32_t n, double *L, int64_t ldl, double *B, int64_t ldb, int32_t nrhs,
                           double *work, const int32_t *dinfo, void *stream, std::string &err) {
  if (nrhs <= 0 || n <= 0) return RH_OK;
  static_assert(kNB == 64, "a block of unknowns is a panel");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int32_t last = (n - 1) / kNB * kNB;
  for (int32_t j0 = last; j0 >= 0; j0 -= kNB) {
    const uint32_t groups = (uint32_t)std::max(1, (j0 + kNB - 1) / kNB);
    const double *diag = j0 == last && nrhs > kNB ? diag_of(dinfo, last) : nullptr;
    hipLaunchKernelGGL(chol_back_block, dim3(groups, (uint32_t)nrhs), dim3(256), 0, st, L, ldl, n, B, ldb, work, j0,
                       dinfo, diag);
  }
  const int64_t total = (int64_t)n * nrhs;
  hipLaunchKernelGGL(dense_copy_cols, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, st, (const double *)work,
                     n, B, ldb, nrhs);
  DENSE_TRY(hipGetLastError());
  return RH_OK;
}

rh_status dense_shift_copy(int32_t n, const double *A, int64_t lda, double *F, int64_t ldf, double tau, void *stream,
                           std::string &err) {
  if (n <= 0) return RH_OK;
  hipLaunchKernelGGL(dense_shift_copy, dim3(n), dim3(256), 0, static_cast<hipStream_t>(stream), A, lda, F, ldf, n,
                     tau);
  DENSE_TRY(hipGetLastError());
  return RH_OK;
}

rh_status dense_diagonal(int32_t n, const double *A, int64_t lda, double *out, void *stream, std::string &err) {
  if (n <= 0) return RH_OK;
  hipLaunchKernelGGL(dense_diag, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream), A, lda, n,
                     out);
  DENSE_TRY(hipGetLastError());
  return RH_OK;
}

rh_status dense_negate(int32_t n, const double *a, double *b, void *stream, std::string &err) {
  if (n <= 0) return RH_OK;
  hipLaunchKernelGGL(dense_neg, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream), a, b, n);
  DENSE_TRY(hipGetLastError());
  return RH_OK;
}

}  // namespace rh
