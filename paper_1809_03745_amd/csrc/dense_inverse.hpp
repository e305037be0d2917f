// Dense FP64 inverse of a bottom-level operator on the device (gfx950).
//
// Blocked Gauss-Jordan elimination with partial pivoting, in place up to the
// row order: panels of NB columns are eliminated by one workgroup that keeps
// U whole panel rows per thread in registers (a column costs a key maximum
// and one exchanged row through LDS), the other columns follow in one
// matrix product per panel over the whole chip, from one buffer into the
// other, which also applies the panel's row exchanges. The panels' serial
// columns bound it. Diagonally dominant matrices (plain boxes) need no pivot
// search: their panels cost a fifth (18 us against 84 at n = 512). An
// unblocked elimination on one host core took 35 ms for the 512 unknowns of an
// 8^3 bottom level, most of a served request that brings new coefficients;
// this takes 1.5 ms, and 0.5 ms where no pivots are searched.
#pragma once

#include "block_engine.hpp"

namespace ebmg {

constexpr int kInvThreads = 1024;
constexpr int kInvTile = 64;        // tile of the update product

// A (row-major, n x n) of a level: blocks [0, N) the cells' template or
// identity rows, blocks [N, N + R) the explicit rows.
template <int DIM>
__global__ void __launch_bounds__(256) k_dense_rows(BLev<double> L, double* __restrict__ A) {
  const int n = L.N + L.N2;
  const int blk = blockIdx.x;
  int64_t q;
  if (blk < L.N) {
    q = blk;
    if (tclass(L.tag[blk]) == 2) return;
  } else {
    q = L.irow_dof[blk - L.N];
  }
  double* row = A + q * n;
  for (int c = threadIdx.x; c < n; c += blockDim.x) row[c] = 0.0;
  __syncthreads();
  if (blk >= L.N) {
    const int r = blk - L.N;
    // a row's columns are distinct
    for (int64_t e = L.rp[r] + threadIdx.x; e < L.rp[r + 1]; e += blockDim.x) row[L.col[e]] = L.val[e];
    if (threadIdx.x == 0) row[q] = L.diag[r];
    return;
  }
  if (threadIdx.x != 0) return;
  const int p = tclass(L.tag[blk]);
  if (p == 3) {
    row[q] = 1.0;
    return;
  }
  const int nx = L.n[0], ny = L.n[1], nz = DIM == 3 ? L.n[2] : 1;
  const int i = blk % nx, j = (blk / nx) % ny, k = blk / (nx * ny);
  double dg = L.tp.D0(p);
  const double co = L.tp.CO(p);
  if (i > 0) row[q - 1] = co; else dg += L.tp.CB(0, p);
  if (i < nx - 1) row[q + 1] = co; else dg += L.tp.CB(1, p);
  if (j > 0) row[q - nx] = co; else dg += L.tp.CB(2, p);
  if (j < ny - 1) row[q + nx] = co; else dg += L.tp.CB(3, p);
  if (DIM == 3) {
    if (k > 0) row[q - nx * ny] = co; else dg += L.tp.CB(4, p);
    if (k < nz - 1) row[q + nx * ny] = co; else dg += L.tp.CB(5, p);
  }
  row[q] = dg;
}

// Eliminates columns [k0, k0 + NB) of X, rows r = tid + u * 1024 in registers;
// writes the panel of the transformation to the same columns of Y, the rows'
// places before the panel's exchanges to src, and carries perm (the original
// row at each place) along. A zero pivot raises flag.
template <int NB, int U>
__global__ void __launch_bounds__(kInvThreads) k_inv_panel(const double* __restrict__ X, double* __restrict__ Y,
                                                          int n, int k0, int* __restrict__ src,
                                                          const int* __restrict__ perm_in, int* __restrict__ perm_out,
                                                          int* __restrict__ flag) {
  static_assert(NB * U <= 32, "at most 32 values of the panel per thread");
  __shared__ double prow[2][NB], krow[2][NB];
  __shared__ int sidx[2][2];
  __shared__ uint32_t wmax[2][kInvThreads / 64];
  const int tid = threadIdx.x;
  const int nb = min(NB, n - k0);
  double a[U][NB];
  int from[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int r = tid + u * kInvThreads;
    from[u] = r;
#pragma unroll
    for (int c = 0; c < NB; ++c) a[u][c] = r < n && c < nb ? X[(int64_t)r * n + k0 + c] : 0.0;
  }
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    if (c < nb) {
      const int kc = k0 + c, buf = c & 1;
      // the largest magnitude at or below the diagonal (by its leading 20 bits;
      // the lowest row among equals)
      uint32_t key = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = tid + u * kInvThreads;
        const uint32_t hi = (uint32_t)(__double_as_longlong(a[u][c]) >> 32) & 0x7fffffffu;
        if (r >= kc && r < n) key = max(key, (hi & 0xfffff000u) | (uint32_t)(4095 - r));
      }
      for (int o = 32; o > 0; o >>= 1) key = max(key, (uint32_t)__shfl_xor((int)key, o, 64));
      if ((tid & 63) == 0) wmax[buf][tid >> 6] = key;
      __syncthreads();
      key = wmax[buf][0];
#pragma unroll
      for (int w = 1; w < kInvThreads / 64; ++w) key = max(key, wmax[buf][w]);
      const int pr = 4095 - (int)(key & 4095u);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = tid + u * kInvThreads;
        if (r == pr) {
#pragma unroll
          for (int j = 0; j < NB; ++j) prow[buf][j] = a[u][j];
          sidx[buf][0] = from[u];
        }
        if (r == kc) {
#pragma unroll
          for (int j = 0; j < NB; ++j) krow[buf][j] = a[u][j];
          sidx[buf][1] = from[u];
        }
      }
      __syncthreads();
      const double pivot = prow[buf][c];
      if (tid == 0 && !(pivot != 0.0)) *flag = 1;
      const double pv = 1.0 / pivot;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = tid + u * kInvThreads;
        if (r == pr) {
#pragma unroll
          for (int j = 0; j < NB; ++j) a[u][j] = krow[buf][j];
          from[u] = sidx[buf][1];
        }
        if (r == kc) {
#pragma unroll
          for (int j = 0; j < NB; ++j) a[u][j] = j == c ? pv : prow[buf][j] * pv;
          from[u] = sidx[buf][0];
        } else {
          const double f = a[u][c];
#pragma unroll
          for (int j = 0; j < NB; ++j) a[u][j] = (j == c ? 0.0 : a[u][j]) - f * (j == c ? pv : prow[buf][j] * pv);
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int r = tid + u * kInvThreads;
    if (r >= n) continue;
#pragma unroll
    for (int c = 0; c < NB; ++c)
      if (c < nb) Y[(int64_t)r * n + k0 + c] = a[u][c];
    src[r] = from[u];
    perm_out[r] = perm_in ? perm_in[from[u]] : from[u];
  }
}

// The same panel without exchanges, for a diagonally dominant matrix (the
// pivots then stay the diagonal's and no entry grows beyond twice the largest):
// only the NB x NB diagonal block is eliminated column by column, one thread an
// entry, by every workgroup for itself, and each takes its share of the panel's
// rows as a product with the block's inverse. The panel above passes all n rows
// through each column (2.6 us a column at n = 512: 84 us a panel).
template <int NB>
__global__ void __launch_bounds__(NB * NB) k_inv_panel_dd(const double* __restrict__ X, double* __restrict__ Y, int n,
                                                        int k0, int* __restrict__ src, int* __restrict__ perm,
                                                        int* __restrict__ flag) {
  __shared__ double prow[2][NB], pcol[2][NB], S[NB][NB + 1], XR[NB][NB + 1];
  const int i = threadIdx.x / NB, j = threadIdx.x % NB;
  const int nb = min(NB, n - k0);
  const int r = blockIdx.x * NB + i;   // the panel row of this thread
  XR[i][j] = r < n && j < nb ? X[(int64_t)r * n + k0 + j] : 0.0;
  double v = i < nb && j < nb ? X[(int64_t)(k0 + i) * n + k0 + j] : (i == j ? 1.0 : 0.0);
  for (int c = 0; c < nb; ++c) {
    const int buf = c & 1;
    if (i == c) prow[buf][j] = v;
    if (j == c) pcol[buf][i] = v;
    __syncthreads();
    const double pivot = prow[buf][c];
    if (blockIdx.x == 0 && threadIdx.x == 0 && !(pivot != 0.0)) *flag = 1;
    const double pv = 1.0 / pivot;
    const double row = j == c ? pv : prow[buf][j] * pv;
    v = i == c ? row : (j == c ? 0.0 : v) - pcol[buf][i] * row;
  }
  S[i][j] = v;
  __syncthreads();
  if (r >= n) return;
  double e = 0.0;
  if (r >= k0 && r < k0 + nb) {
    e = S[r - k0][j];
  } else {
#pragma unroll 8
    for (int c = 0; c < NB; ++c) e -= XR[i][c] * S[c][j];
  }
  if (j < nb) Y[(int64_t)r * n + k0 + j] = e;
  if (j == 0) {
    src[r] = r;
    perm[r] = r;
  }
}

// The other columns: Y[i][j] = (i in the panel ? 0 : X[src i][j]) +
// sum_c E[i][c] X[src (k0 + c)][j], E the panel columns of Y.
template <int NB>
__global__ void __launch_bounds__(256) k_inv_update(const double* __restrict__ X, double* __restrict__ Y, int n,
                                                   int k0, const int* __restrict__ src) {
  constexpr int TM = kInvTile;
  __shared__ double E[NB][TM + 1], B[NB][TM];
  const int nb = min(NB, n - k0);
  const int i0 = blockIdx.y * TM, j0 = blockIdx.x * TM;
  for (int t = threadIdx.x; t < TM * NB; t += 256) {
    const int c = t % NB, i = t / NB;
    E[c][i] = i0 + i < n && c < nb ? Y[(int64_t)(i0 + i) * n + k0 + c] : 0.0;
    const int j = t % TM, d = t / TM;
    B[d][j] = j0 + j < n && d < nb ? X[(int64_t)src[k0 + d] * n + j0 + j] : 0.0;
  }
  __syncthreads();
  const int tj = (threadIdx.x & 15) * 4, ti = (threadIdx.x >> 4) * 4;
  double acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int i = i0 + ti + a;
    const bool keep = i < n && !(i >= k0 && i < k0 + nb);
    const int64_t base = keep ? (int64_t)src[i] * n : 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = keep && j0 + tj + b < n ? X[base + j0 + tj + b] : 0.0;
  }
#pragma unroll 4
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double e = E[c][ti + a];
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] += e * B[c][tj + b];
    }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = i0 + ti + a, j = j0 + tj + b;
      if (i < n && j < n && !(j >= k0 && j < k0 + nb)) Y[(int64_t)i * n + j] = acc[a][b];
    }
}

// Ainv[i][perm[j]] = X[i][j]
__global__ void __launch_bounds__(256) k_inv_columns(const double* __restrict__ X, double* __restrict__ Ainv, int n,
                                                     const int* __restrict__ perm) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * n) return;
  const int64_t i = t / n;
  const int j = (int)(t % n);
  Ainv[i * n + perm[j]] = X[t];
}

}  // namespace ebmg
