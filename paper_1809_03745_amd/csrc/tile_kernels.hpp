// One side of a V-cycle on a small level in one launch: the pre-smoothing
// from zero with the residual and its restriction, or the prolongation with
// the post-smoothing.
//
// Small levels are bound by the number of dependent launches, not by bytes:
// a V(2,2) level took eleven of them (eight colour phases, residual,
// restriction, prolongation). Here a workgroup holds one tile of the level
// with a halo on each side in LDS and does all phases there, updating as the
// out-of-place colour phases do (k_rb_oop); a phase moves information by one
// cell, or the reach of a row, so after four phases (or three and the
// residual, the first one starting from zero) every value in the tile itself
// is the one the phase-by-phase launches give, and only halo cells, which are
// dropped, are stale. The halo is computed again by the neighbour:
// 1.8 to 2.6 times the work in 2D (24 x 24 of 32 x 32, 40 x 40 of 64 x 64) and
// eight times in 3D (8^3 of 16^3), which is why the rule of use ends at small
// levels. The halo is four times the reach of the level's explicit rows; in
// 3D only rows that read their 26 neighbours fit.
//
// A launch waits on latency: about 4 us to start, three dependent loads (the
// tile's list, its rows, their values), then 0.6 us a phase; 8 to 11 us at
// 16^3, 32^3 and 32^2 to 256^2 (12 to 18 us at 16^3 and 32^3 with the rows of a
// pin, 28 us at 64^3). Row entries held in registers over the phases
// did not change it (they come from L2 while the template cells compute).
// Two 1024-thread workgroups fit a CU where the launch bounds say so, 33 -> 26
// us at 1024^2. Bounds are set so that nothing spills.
// A 1024^2 two-disk solve in FP64: 8.4 -> 4.1 ms; a 128^3 box: 2.40 -> 2.08 ms.
#pragma once

#include "kernels.hpp"

namespace ebmg {

constexpr int kTilePhases = 4;    // phases a launch may advance
constexpr int kTileRows = 1024;   // explicit rows a tile and its halo may hold
constexpr int kTileLanes = 4;     // lanes that share an explicit row
// H: halo on each side, kTilePhases times the reach of the level's rows
template <int DIM, int H>
struct TileDim {
  static constexpr int E = DIM == 3 ? 16 : H == 4 ? 32 : H == 8 ? 48 : 64;   // cells along an axis with the halo
  static constexpr int C = E - 2 * H;                                        // cells of the tile proper
  static constexpr int EZ = DIM == 3 ? E : 1;
  static constexpr int NE = E * E * EZ;
  static constexpr int NT = DIM == 3 ? 1024 : H == 4 ? 512 : H == 8 ? 576 : 1024;   // threads
  static constexpr int NP = NE / 2 / NT;                  // even-odd pairs of a thread
  static constexpr int PAD = DIM == 3 ? E * E : E;        // readable before and after the cells
};

// An explicit row as one tile sees it. loc: its unknown's place in LDS (cells
// first, then second-phase unknowns by their row's place in the tile's list);
// core: its cell lies in the tile proper.
struct TileRow {
  int32_t beg;    // first entry in the level's row values
  int32_t lcol;   // first entry in the tile's local columns
  uint32_t bits;  // loc | entries << 13 | core << 31
  int32_t dof;
};

template <typename T>
struct TileView {
  Tmpl<T> tp;
  int cn[3], nt[3];
  const uint8_t *tag, *ctag;
  const T *val, *diag;
  // per tile t: rows [ptr[2t], ptr[2t + 1]) of group 0 and up to ptr[2t + 2] of group 1
  const int32_t* ptr;
  const TileRow* row;
  const int32_t* rid;       // row of the level (its diagonal)
  const uint16_t* lcol;     // places in LDS, 0 where a column lies outside (such rows are stale)
  // fine unknowns of non-simple parents, by tile with halo
  const int32_t* npp;
  const uint16_t* npl;
  const int32_t* npc;
  // non-simple coarse unknowns, by tile, and their children's places
  const int32_t *nsp, *nsd, *nsq;
  const uint16_t* nsl;
};

// reciprocal diagonal of a template cell of phase p (as the smoother kernels form it)
template <typename T, int DIM>
__device__ __forceinline__ T tile_rdiag(const Tmpl<T>& tp, int p, int i, int j, int k) {
  if (p > 1) return T(0);
  T dg = tp.D0(p);
  if (!(i > 0)) dg += tp.CB(0, p);
  if (!(i < tp.n[0] - 1)) dg += tp.CB(1, p);
  if (!(j > 0)) dg += tp.CB(2, p);
  if (!(j < tp.n[1] - 1)) dg += tp.CB(3, p);
  if (DIM == 3) {
    if (!(k > 0)) dg += tp.CB(4, p);
    if (!(k < tp.n[2] - 1)) dg += tp.CB(5, p);
  }
  return T(1) / dg;
}

// PRE: x = 0, `phases` colour phases, xo = x, bc = restriction of b - A x.
// else: x = xin + P ec, `phases` colour phases, xo = x (add: xo += x).
template <typename T, int DIM, int H, bool PRE, bool ROWS>
__global__ void __launch_bounds__((TileDim<DIM, H>::NT), (H == 12 || (DIM == 3 && !ROWS) ? 8 : 4)) k_tile(TileView<T> V, const T* __restrict__ xin,
                                                           const T* __restrict__ ec, const T* __restrict__ b,
                                                           T* __restrict__ xo, T* __restrict__ bc, int phases,
                                                           bool add) {
  using D = TileDim<DIM, H>;
  constexpr int E = D::E, NT = D::NT, NP = D::NP, PAD = D::PAD, HX = E / 2;
  constexpr int RM = ROWS ? kTileRows : 1;
  __shared__ T xs_[PAD + D::NE + (ROWS ? kTileRows : 0) + PAD];
  __shared__ T rb[RM], rd[RM], rv[RM];
  __shared__ int32_t rbeg[RM], rcol[RM];
  __shared__ uint32_t rbit[RM];
  T* const xs = xs_ + PAD;
  const Tmpl<T>& tp = V.tp;
  const int nx = tp.n[0], ny = tp.n[1], nz = DIM == 3 ? tp.n[2] : 1;
  const int t = (int)threadIdx.x, tile = (int)blockIdx.x;
  const int ti = tile % V.nt[0], tjk = tile / V.nt[0];
  const int tj = DIM == 3 ? tjk % V.nt[1] : tjk, tk = DIM == 3 ? tjk / V.nt[1] : 0;
  const int oi = ti * D::C - H, oj = tj * D::C - H, ok = DIM == 3 ? tk * D::C - H : 0;

  // cells of the tile: NP even-odd pairs a thread
  T xq[NP][2], bq[NP][2], rdg[NP][2];   // right-hand side and reciprocal diagonal
  uint32_t cls = 0;                     // classes, four bits a cell (4: outside the box)
  auto cl = [&](int s, int u) { return (int)((cls >> (8 * s + 4 * u)) & 15u); };
  const int li = 2 * (t % HX), lj0 = t / HX;
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int jk = lj0 + s * (NT / HX);
    const int lj = DIM == 3 ? jk % E : jk, lk = DIM == 3 ? jk / E : 0;
    const int i = oi + li, j = oj + lj, k = ok + lk;
    const bool in = i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz;
    const int c = in ? i + nx * (j + ny * k) : 0;
    T e = 0;
    bool up = false;
    if (!PRE && in) {
      const int P = (i >> 1) + V.cn[0] * ((j >> 1) + V.cn[1] * (k >> 1));
      e = ec[P];
      up = !(V.ctag[P] & 4);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool inu = in && i + u < nx;
      const int p = inu ? (int)tclass(V.tag[c + u]) : 4;
      cls |= (uint32_t)p << (8 * s + 4 * u);
      bq[s][u] = inu ? b[c + u] : T(0);
      rdg[s][u] = tile_rdiag<T, DIM>(tp, p, i + u, j, k);
      T v = 0;
      if (!PRE && inu) {
        v = xin[c + u];
        if (p != 3 && up) v = v + e;
      }
      xq[s][u] = v;
    }
  }
  // rows of the tile; the first transfer entry of each thread is taken here
  // too, so that all loads of the launch wait together
  int g1 = 0, nr = 0, t0 = 0, t1 = 0;
  const TileRow* rows = nullptr;
  int npl = 0;
  T npe = 0;
  if (ROWS) {
    const int r0 = V.ptr[2 * tile];
    g1 = V.ptr[2 * tile + 1] - r0;
    nr = V.ptr[2 * tile + 2] - r0;
    rows = V.row + r0;
    t0 = (PRE ? V.nsp : V.npp)[tile];
    t1 = (PRE ? V.nsp : V.npp)[tile + 1];
    if (!PRE && t0 + t < t1) {
      npl = V.npl[t0 + t];
      npe = ec[V.npc[t0 + t]];
    }
    for (int q = t; q < nr; q += NT) {
      const TileRow w = rows[q];
      rbeg[q] = w.beg;
      rcol[q] = w.lcol;
      rbit[q] = w.bits;
      rb[q] = b[w.dof];
      rd[q] = V.diag[V.rid[r0 + q]];
      const int loc = (int)(w.bits & 8191u);
      if (loc >= D::NE) xs[loc] = PRE ? T(0) : xin[w.dof];
    }
  }
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int jk = lj0 + s * (NT / HX);
    xs[li + E * jk] = xq[s][0];
    xs[li + 1 + E * jk] = xq[s][1];
  }
  for (int q = t; q < PAD; q += NT) {
    xs_[q] = T(0);
    xs[D::NE + (ROWS ? kTileRows : 0) + q] = T(0);
  }
  __syncthreads();
  if (!PRE && ROWS) {
    if (t0 + t < t1) xs[npl] += npe;
    for (int q = t0 + t + NT; q < t1; q += NT) xs[V.npl[q]] += ec[V.npc[q]];
    __syncthreads();
  }

  auto dot = [&](int q) {   // off-diagonal sum of row q, by kTileLanes lanes
    const int n = (int)((rbit[q] >> 13) & 0x3ffffu);
    const T* va = V.val + rbeg[q];
    const uint16_t* co = V.lcol + rcol[q];
    T s = 0;
#pragma unroll 2
    for (int e = t % kTileLanes; e < n; e += kTileLanes) s += va[e] * xs[co[e]];
    for (int off = kTileLanes / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kTileLanes);
    return s;
  };
  for (int ph = 0; ph < phases; ++ph) {
    const int colour = ph & 1;
    if (ROWS) {
      const int q1 = colour ? nr : g1;
      for (int q = (colour ? g1 : 0) + t / kTileLanes; q < q1; q += NT / kTileLanes) {
        const T s = PRE && ph == 0 ? T(0) : dot(q);
        if (t % kTileLanes == 0) rv[q] = (rb[q] - s) / rd[q];
      }
    }
    T nv[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int jk = lj0 + s * (NT / HX);
      const int i = oi + li, j = oj + (DIM == 3 ? jk % E : jk), k = DIM == 3 ? ok + jk / E : 0;
      const int u = ((i + j + k) & 1) == colour ? 0 : 1;
      const int m = li + u + E * jk;
      const int p = cl(s, u);
      nv[s] = xs[m];
      if (p <= 1) {
        T sm = 0;
        if (!PRE || ph > 0) {   // (the first phase from zero reads nothing: good up to the halo's edge)
          const int iu = i + u;
          if (iu > 0) sm += xs[m - 1];
          if (iu < nx - 1) sm += xs[m + 1];
          if (j > 0) sm += xs[m - E];
          if (j < ny - 1) sm += xs[m + E];
          if (DIM == 3) {
            if (k > 0) sm += xs[m - E * E];
            if (k < nz - 1) sm += xs[m + E * E];
          }
        }
        nv[s] = tmpl_update_r<T>(tp, p, u ? bq[s][1] : bq[s][0], sm, u ? rdg[s][1] : rdg[s][0]);
      }
    }
    if (ROWS) __syncthreads();   // explicit rows read this colour's cells as they were
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const int jk = lj0 + s * (NT / HX);
      const int i = oi + li, j = oj + (DIM == 3 ? jk % E : jk), k = DIM == 3 ? ok + jk / E : 0;
      const int u = ((i + j + k) & 1) == colour ? 0 : 1;
      if (cl(s, u) <= 1) xs[li + u + E * jk] = nv[s];
    }
    if (ROWS) {
      const int q1 = colour ? nr : g1;
      for (int q = (colour ? g1 : 0) + t; q < q1; q += NT) xs[rbit[q] & 8191u] = rv[q];
    }
    __syncthreads();
  }

  // the tile's values out, and its residual
  T rq[NP][2];
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int jk = lj0 + s * (NT / HX);
    const int lj = DIM == 3 ? jk % E : jk, lk = DIM == 3 ? jk / E : 0;
    const int i = oi + li, j = oj + lj, k = ok + lk;
    const bool core = li >= H && li < E - H && lj >= H && lj < E - H &&
                      (DIM < 3 || (lk >= H && lk < E - H));
    const int c = i + nx * (j + ny * k);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = li + u + E * jk, p = cl(s, u);
      rq[s][u] = 0;
      if (!core || p == 4) continue;
      const T xv = xs[m];
      xo[c + u] = !PRE && add ? xo[c + u] + xv : xv;
      if (PRE && p <= 1) {
        T sm = 0;
        T dg = tp.M(p);
        if (i + u > 0) sm += xs[m - 1] - xv; else dg += tp.CBM(0, p);
        if (i + u < nx - 1) sm += xs[m + 1] - xv; else dg += tp.CBM(1, p);
        if (j > 0) sm += xs[m - E] - xv; else dg += tp.CBM(2, p);
        if (j < ny - 1) sm += xs[m + E] - xv; else dg += tp.CBM(3, p);
        if (DIM == 3) {
          if (k > 0) sm += xs[m - E * E] - xv; else dg += tp.CBM(4, p);
          if (k < nz - 1) sm += xs[m + E * E] - xv; else dg += tp.CBM(5, p);
        }
        rq[s][u] = bq[s][u] - (dg * xv + tp.CO(p) * sm);
      }
    }
  }
  if (ROWS) {
    // second-phase unknowns out
    for (int q = t; q < nr; q += NT) {
      const int loc = (int)(rbit[q] & 8191u);
      if (loc >= D::NE && (rbit[q] >> 31)) {
        T* o = xo + rows[q].dof;
        *o = !PRE && add ? *o + xs[loc] : xs[loc];
      }
    }
  }
  if (!PRE) return;
  if (ROWS) {
    for (int q = t / kTileLanes; q < nr; q += NT / kTileLanes) {
      const uint32_t w = rbit[q];
      if (!(w >> 31)) continue;
      const T s = dot(q);
      if (t % kTileLanes == 0) rv[q] = rb[q] - (rd[q] * xs[w & 8191u] + s);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int jk = lj0 + s * (NT / HX);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (cl(s, u) != 2) xs[li + u + E * jk] = rq[s][u];
  }
  if (ROWS)
    for (int q = t; q < nr; q += NT)
      if (rbit[q] >> 31) xs[rbit[q] & 8191u] = rv[q];
  __syncthreads();
  // restriction: mean of the children of the tile's simple coarse cells (0 in
  // covered ones), and the non-simple coarse unknowns' lists
  constexpr int CC = D::C / 2;
  const T w = DIM == 3 ? T(0.125) : T(0.25);
  if (t < CC * CC * (DIM == 3 ? CC : 1)) {
    const int a = t % CC, q = t / CC;
    const int ai = a, aj = DIM == 3 ? q % CC : q, ak = DIM == 3 ? q / CC : 0;
    const int I = ti * CC + ai, J = tj * CC + aj, K = DIM == 3 ? tk * CC + ak : 0;
    if (I < V.cn[0] && J < V.cn[1] && (DIM < 3 || K < V.cn[2])) {
      const int P = I + V.cn[0] * (J + V.cn[1] * K);
      const uint8_t tg = V.ctag[P];
      const int m = H + 2 * ai + E * (H + 2 * aj + (DIM == 3 ? E * (H + 2 * ak) : 0));
      if (tclass(tg) == 3) {
        bc[P] = 0;
      } else if (!(tg & 4)) {
        T s = xs[m] + xs[m + 1] + xs[m + E] + xs[m + E + 1];
        if (DIM == 3) s += xs[m + E * E] + xs[m + E * E + 1] + xs[m + E * E + E] + xs[m + E * E + E + 1];
        bc[P] = s * w;
      }
    }
  }
  if (ROWS) {
    constexpr int NC = DIM == 3 ? 8 : 4;   // children whose loads go out together
    for (int q = t0 + t; q < t1; q += NT) {
      const int e0 = V.nsq[q], n = V.nsq[q + 1] - e0;
      const uint16_t* m = V.nsl + e0;
      int l[NC];
#pragma unroll
      for (int e = 0; e < NC; ++e) l[e] = e < n ? (int)m[e] : 0;
      T s = 0;
#pragma unroll
      for (int e = 0; e < NC; ++e)
        if (e < n) s += xs[l[e]];
      for (int e = NC; e < n; ++e) s += xs[m[e]];
      bc[V.nsd[q]] = s * w;
    }
  }
}

}  // namespace ebmg
