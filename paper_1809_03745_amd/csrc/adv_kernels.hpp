// One explicit advection step of a density on the gas phase of a cut-cell
// grid (Convection-Diffusion-Reaction equations: Advective discretization,
// Hybrid divergence), FP64:
//   k_adv_rows     (3D) the two launches below fused into one z-marching
//                  pass over the box;
//   k_adv_flux     face-centred fluxes u n_f of one direction, n_f the
//                  upwind state of an unsplit Godunov predictor with
//                  monotonised-central (van Leer) slopes, extrapolated to the
//                  face and to the half step including the transverse terms;
//                  inflow domain faces take the boundary density;
//   k_adv_full     full cells (every face full: the centroid fluxes are the
//                  face-centred ones): conservative divergence and
//                  n_out = n - dt D^c; 0 where there is no gas;
//   k_adv_dc_cut   conservative divergence of cut cells from their
//                  precomputed forms over the face fluxes (apertures,
//                  centroid interpolation, 1 / (kappa h));
//   k_adv_cut      per cut cell: the non-conservative divergence (kappa-
//                  weighted mean over its 3^D block), the hybrid
//                  kappa D^c + (1 - kappa) D^nc, and the rate change
//                  dM / S its mass defect dM = kappa (1 - kappa)(D^nc - D^c)
//                  gives every other gas cell of its block;
//   k_adv_special  cut cells and the cells receiving redistributed mass:
//                  n_out = n - dt (their hybrid or D^c, less what they
//                  receive), overwriting the previous launch's value.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace ebmg {

constexpr int kAdvX = 60;   // cells of a row a wavefront of k_adv_rows completes

struct AdvGrid {
  int n[3];
  int dim;
  int64_t fbase[3];
  double h, dt;
  double inflow[6];
};

// sign of the differences times min(2 |dl|, 2 |dr|, |dl + dr| / 2), 0 unless
// they have the same sign
__device__ __forceinline__ double adv_mc(double dl, double dr) {
  const double m = fmin(fabs(dl), fabs(dr)), s = dl + dr;
  const double v = __builtin_copysign(fmin(2.0 * m, fabs(0.5 * s)), s);
  return dl * dr > 0.0 ? v : 0.0;
}

template <int DIM>
__device__ __forceinline__ bool adv_gas(const uint8_t* __restrict__ cls, const AdvGrid& G, int i, int j, int k) {
  if (i < 0 || i >= G.n[0] || j < 0 || j >= G.n[1]) return false;
  if (DIM == 3 && (k < 0 || k >= G.n[2])) return false;
  return cls[i + (int64_t)G.n[0] * (j + (int64_t)G.n[1] * k)] != 0;
}

// slope of cell (i, j, k) along e (0 without gas on both sides)
template <int DIM>
__device__ __forceinline__ double adv_slope(const double* __restrict__ n, const uint8_t* __restrict__ cls,
                                            const AdvGrid& G, int i, int j, int k, int e) {
  const int di = e == 0, dj = e == 1, dk = e == 2;
  if (!adv_gas<DIM>(cls, G, i - di, j - dj, k - dk) || !adv_gas<DIM>(cls, G, i + di, j + dj, k + dk)) return 0.0;
  const int64_t sx = 1, sy = G.n[0], sz = (int64_t)G.n[0] * G.n[1];
  const int64_t c = i + sy * j + sz * k;
  const int64_t st = e == 0 ? sx : (e == 1 ? sy : sz);
  const double nc = n[c];
  return adv_mc(nc - n[c - st], n[c + st] - nc);
}

// face velocity of direction e at face index (fi, fj, fk)
template <int DIM>
__device__ __forceinline__ double adv_u(const double* const* u, const AdvGrid& G, int e, int fi, int fj, int fk) {
  const int64_t m0 = G.n[0] + (e == 0), m1 = G.n[1] + (e == 1);
  return u[e][fi + m0 * (fj + m1 * (int64_t)fk)];
}

struct AdvVel {
  const double* u[3];
};

// flux u n_f through face (fi, fj, fk) of direction DIR (face index along
// DIR = the index of its high cell), read from global memory
template <int DIM, int DIR>
__device__ __forceinline__ double adv_face_flux(const double* __restrict__ n, const uint8_t* __restrict__ cls,
                                                const AdvVel& vel, const AdvGrid& G, int fi, int fj, int fk) {
  const int m0 = G.n[0] + (DIR == 0), m1 = G.n[1] + (DIR == 1);
  const int64_t fl = fi + (int64_t)m0 * (fj + (int64_t)m1 * fk);
  const int fc[3] = {fi, fj, fk};
  const double u = vel.u[DIR][fl];
  const double h = G.h, dt = G.dt;
  const bool up_lo = u >= 0.0;
  // the upwind cell: the low one (face on its high side) or the high one
  int c[3] = {fi, fj, fk};
  if (up_lo) c[DIR] -= 1;
  const bool outside = up_lo ? fc[DIR] == 0 : fc[DIR] == G.n[DIR];
  if (outside) return u * G.inflow[2 * DIR + (up_lo ? 0 : 1)];
  if (!adv_gas<DIM>(cls, G, c[0], c[1], c[2])) return 0.0;
  const int64_t cc = c[0] + (int64_t)G.n[0] * (c[1] + (int64_t)G.n[1] * c[2]);
  double trans = 0.0;
#pragma unroll
  for (int e = 0; e < DIM; ++e) {
    if (e == DIR) continue;
    int hi[3] = {c[0], c[1], c[2]};
    hi[e] += 1;
    const double ve = 0.5 * (adv_u<DIM>(vel.u, G, e, c[0], c[1], c[2]) + adv_u<DIM>(vel.u, G, e, hi[0], hi[1], hi[2]));
    trans += ve * adv_slope<DIM>(n, cls, G, c[0], c[1], c[2], e);
  }
  const double base = n[cc] - 0.5 * dt / h * trans;
  const double sd = adv_slope<DIM>(n, cls, G, c[0], c[1], c[2], DIR);
  return u * (base + ((up_lo ? 0.5 : -0.5) - u * dt / (2.0 * h)) * sd);
}

// one direction's face fluxes: thread = face of one z plane (x fastest),
// blockIdx.y = the face's z index; F is that direction's face array
template <int DIM, int DIR>
__global__ void __launch_bounds__(256) k_adv_flux(const double* __restrict__ n, const uint8_t* __restrict__ cls,
                                                  AdvVel vel, AdvGrid G, double* __restrict__ F) {
  const unsigned m0 = G.n[0] + (DIR == 0), m1 = G.n[1] + (DIR == 1);
  const unsigned f2 = blockIdx.x * 256u + threadIdx.x;
  if (f2 >= m0 * m1) return;
  const int fk = DIM == 3 ? (int)blockIdx.y : 0;
  F[f2 + (int64_t)m0 * m1 * fk] = adv_face_flux<DIM, DIR>(n, cls, vel, G, (int)(f2 % m0), (int)(f2 / m0), fk);
}

// cells with every face full (class 1, or 3 when a cut cell's block needs
// their D^c): n_out = n - dt D^c; cells without gas get 0; cut cells are
// left to the cut-cell launches. Thread = cell of one z plane.
template <int DIM>
__global__ void __launch_bounds__(256) k_adv_full(const uint8_t* __restrict__ cls, AdvGrid G,
                                                  const double* __restrict__ F, const double* __restrict__ n,
                                                  double* __restrict__ Dc, double* __restrict__ nout) {
  const unsigned nx = G.n[0], ny = G.n[1];
  const unsigned c2 = blockIdx.x * 256u + threadIdx.x;
  if (c2 >= nx * ny) return;
  const int k = DIM == 3 ? (int)blockIdx.y : 0;
  const int64_t c = c2 + (int64_t)nx * ny * k;
  const uint8_t t = cls[c];
  if (t == 2) return;
  if (t == 0) {
    nout[c] = 0.0;
    return;
  }
  const int i = (int)(c2 % nx), j = (int)(c2 / nx);
  double net = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const int64_t m0 = nx + (d == 0), m1 = ny + (d == 1);
    const int64_t lo = G.fbase[d] + i + m0 * (j + m1 * (int64_t)k);
    const int64_t st = d == 0 ? 1 : (d == 1 ? m0 : m0 * m1);
    net += F[lo + st] - F[lo];
  }
  const double dc = net / G.h;
  if (t == 3) Dc[c] = dc;
  nout[c] = n[c] - G.dt * dc;
}

// The two cut-cell launches give each cut cell kSub lanes over its list (the
// lists of neighbouring cells follow each other, so a wavefront's loads are
// contiguous; one thread per cell took 21 and 29 us for the 69,000 cut cells
// of a 256^3 pin-plane box).
__device__ __forceinline__ double adv_list_sum(int64_t b, int64_t e, const double* __restrict__ coef,
                                               const int64_t* __restrict__ idx, const double* __restrict__ v) {
  double s = 0.0;
  for (int64_t q = b + threadIdx.x % kSub; q < e; q += kSub) s += coef[q] * v[idx[q]];
  for (int off = kSub / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kSub);
  return s;
}

__global__ void __launch_bounds__(256) k_adv_dc_cut(int ncut, const int64_t* __restrict__ cell,
                                                    const int64_t* __restrict__ ptr, const int64_t* __restrict__ face,
                                                    const double* __restrict__ coef, const double* __restrict__ F,
                                                    double* __restrict__ Dc) {
  const int q = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kSub);
  if (q >= ncut) return;
  const double s = adv_list_sum(ptr[q], ptr[q + 1], coef, face, F);
  if (threadIdx.x % kSub == 0) Dc[cell[q]] = s;
}

__global__ void __launch_bounds__(256) k_adv_cut(int ncut, const int64_t* __restrict__ cell,
                                                 const double* __restrict__ kappa, const int64_t* __restrict__ ptr,
                                                 const int64_t* __restrict__ nbc, const double* __restrict__ nbw,
                                                 const double* __restrict__ S, const double* __restrict__ Dc,
                                                 double* __restrict__ Dcut, double* __restrict__ give) {
  const int q = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kSub);
  if (q >= ncut) return;
  const int64_t c = cell[q];
  const double dc = Dc[c], sq = S[q], k = kappa[c];
  const double dnc = adv_list_sum(ptr[q], ptr[q + 1], nbw, nbc, Dc);
  if (threadIdx.x % kSub != 0) return;
  // without a gas neighbour the conservative divergence stays
  Dcut[q] = sq > 0.0 ? k * dc + (1.0 - k) * dnc : dc;
  give[q] = sq > 0.0 ? k * (1.0 - k) * (dnc - dc) / sq : 0.0;
}

__global__ void __launch_bounds__(256) k_adv_special(int nsp, const int64_t* __restrict__ cell,
                                                     const int32_t* __restrict__ cut, const int64_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ donor, double dt,
                                                     const double* __restrict__ n, const double* __restrict__ Dc,
                                                     const double* __restrict__ Dcut, const double* __restrict__ give,
                                                     double* __restrict__ nout) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nsp) return;
  const int64_t c = cell[s];
  double D = cut[s] >= 0 ? Dcut[cut[s]] : Dc[c];
  for (int64_t e = ptr[s]; e < ptr[s + 1]; ++e) D -= give[donor[e]];
  nout[c] = n[c] - dt * D;
}


// value of the lane below / above (0 in lane 0 / 63)
__device__ __forceinline__ double lane_below(double v) {
  const long long b = __double_as_longlong(v);
  const int l = __builtin_amdgcn_mov_dpp((int)b, 0x138, 0xf, 0xf, true);   // wavefront shift right by one
  const int h = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double(((long long)h << 32) | (unsigned)l);
}
__device__ __forceinline__ double lane_above(double v) {
  const long long b = __double_as_longlong(v);
  const int l = __builtin_amdgcn_mov_dpp((int)b, 0x130, 0xf, 0xf, true);   // wavefront shift left by one
  const int h = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x130, 0xf, 0xf, true);
  return __longlong_as_double(((long long)h << 32) | (unsigned)l);
}
// entry at byte offset o (scalar base, 32-bit lane offset)
template <typename T>
__device__ __forceinline__ T& at(T* p, unsigned o) {
  return *(T*)((const char*)p + o);
}

// The whole full-cell step in one pass over the box (3D): a wavefront holds
// 64 consecutive cells of a row, a block R rows, and marches up ZC planes with
// each lane's own column in registers. Lanes 2 .. 61 of rows 1 .. R - 2 are
// the tile, the others its halo, which the same instructions compute: at plane
// k every lane forms its cell's slopes and extrapolation bases (x neighbours
// from the lanes beside it, y neighbours' densities and the bases and slopes
// of the row below through LDS), then the fluxes of its cell's three low
// faces, the upwind side chosen by selects. A cell's high x flux is the next
// lane's low one; its divergence is closed one plane later, when the low z
// flux above it and, through LDS, the low y flux of the next row are there:
// each face is computed once and one barrier per plane suffices (every LDS
// array alternates between two buffers).
// Cells without gas hold NaN in the difference operands, which adv_mc turns
// into the zero slope of the rule; their own fluxes are 0 by their class.
// Cut cells (class 2) only get their face fluxes stored (the cut-cell launches
// finish them); cells of class 2 or 3 store all six into F for the cut-cell
// forms, class 3 also its D^c. Per face the arithmetic is that of
// adv_face_flux, up to contraction of the transverse sums.
// Bound by instruction issue (163 vector instructions a wavefront and plane,
// 57 % of the launch's cycles at four wavefronts a SIMD) and the loads'
// latency. A form with 16 x 16-cell tiles, whose threads each computed both
// faces of two axes in branches and one wavefront of four the halo, took
// 333 us for 256^3 cells (2.1 TB/s of the 41 B per cell); this one 195 to 204
// us (3.4 to 3.5 TB/s). Unrolled over the roles of the carried planes, without their
// moves, it spilled 75 registers and took 465 us.
template <int R, int ZC>
__global__ void __launch_bounds__(64 * R) k_adv_rows(const double* __restrict__ n, const uint8_t* __restrict__ cls,
                                                    AdvVel vel, AdvGrid G, int tiles_x, int tiles_y,
                                                    double* __restrict__ F, double* __restrict__ Dc,
                                                    double* __restrict__ nout) {
  __shared__ double ln[2][R + 2][64];              // densities of the rows and of the one on either side
  __shared__ double lb[2][R][64], ls[2][R][64];    // y-face bases and slopes
  __shared__ double lf[2][R][64];                  // low y fluxes
  __shared__ unsigned long long lg[2][R];          // gas lanes of a row
  // byte offsets within the block's planes fit in 32 bits (checked by the host)
  const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
  const unsigned sxy = (unsigned)nx * ny;              // plane stride of cells and z faces
  const unsigned sfx = (unsigned)(nx + 1) * ny;        // plane stride of x faces
  const unsigned sfy = (unsigned)nx * (ny + 1);        // plane stride of y faces
  const int64_t t = xcd_block(blockIdx.x, gridDim.x);
  const int tpc = tiles_x * tiles_y;
  const int zc = (int)(t / tpc), r = (int)(t % tpc);
  const int i0 = (r % tiles_x) * kAdvX, j0 = (r / tiles_x) * (R - 2);
  const int z0 = zc * ZC, z1 = min(nz, z0 + ZC);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int i = i0 - 2 + lane, j = j0 - 1 + w;
  const bool in = i >= 0 && i < nx && j >= 0 && j < ny;
  const bool out = lane >= 2 && lane < 2 + kAdvX && w >= 1 && w < R - 1 && in;
  const double h = G.h, dt = G.dt, c1 = 0.5 * dt / h, c2 = dt / (2.0 * h), rh = 1.0 / h;
  // the arrays from the block's first plane on
  const int zb = max(z0 - 2, 0);
  const double* __restrict__ nb = n + (int64_t)sxy * zb;
  const uint8_t* __restrict__ clsb = cls + (int64_t)sxy * zb;
  const double* __restrict__ ux = vel.u[0] + (int64_t)sfx * zb;
  const double* __restrict__ uy = vel.u[1] + (int64_t)sfy * zb;
  const double* __restrict__ uz = vel.u[2] + (int64_t)sxy * zb;
  double* __restrict__ nob = nout + (int64_t)sxy * zb;
  double* __restrict__ Dcb = Dc + (int64_t)sxy * zb;
  double* __restrict__ Fx = F + G.fbase[0] + (int64_t)sfx * zb;
  double* __restrict__ Fy = F + G.fbase[1] + (int64_t)sfy * zb;
  double* __restrict__ Fz = F + G.fbase[2] + (int64_t)sxy * zb;
  // in-plane offsets, clamped into the arrays: of the cell, its low x face
  // (one past the box too), its low y face and the next row's
  auto clamp = [](int v, int hi) { return (unsigned)min(max(v, 0), hi); };
  const unsigned oc = clamp(i, nx - 1) + (unsigned)nx * clamp(j, ny - 1);
  const unsigned ox = clamp(i, nx) + (unsigned)(nx + 1) * clamp(j, ny - 1);
  const unsigned oy = clamp(i, nx - 1) + (unsigned)nx * clamp(j, ny);
  const unsigned oyh = clamp(i, nx - 1) + (unsigned)nx * clamp(j + 1, ny);
  // the row beyond the block that the first and the last row difference with
  const bool outer = w == 0 || w == R - 1;
  const int jo = w == 0 ? j - 1 : j + 1;
  const int wo = w == 0 ? 0 : R + 1;
  const bool ino = i >= 0 && i < nx && jo >= 0 && jo < ny;
  const unsigned oo = clamp(i, nx - 1) + (unsigned)nx * clamp(jo, ny - 1);
  const double kNaN = __builtin_nan("");
  const double inx0 = G.inflow[0], inx1 = G.inflow[1], iny0 = G.inflow[2], iny1 = G.inflow[3];
  const double inz0 = G.inflow[4], inz1 = G.inflow[5];
  const bool edge = i0 < 2 || i0 + kAdvX + 2 > nx || j0 < 1 || j0 + R - 1 > ny;
  // requested densities and classes (of the outer row too) and low velocities
  // of a plane; two requests of each are in flight, taken up two steps after
  // they were issued (one step is shorter than a loaded memory's latency)
  struct Den {
    double v, o;
    uint8_t c, oc;
  };
  struct Vlow {
    double x, y, yh, zh;
  };
  auto load_n = [&](int k, Den& d) {
    const unsigned p = sxy * (clamp(k, nz - 1) - zb);
    d.v = at(nb, 8 * (p + oc));
    d.c = at(clsb, p + oc);
    if (outer) {
      d.o = at(nb, 8 * (p + oo));
      d.oc = at(clsb, p + oo);
    }
  };
  auto load_u = [&](int k, Vlow& v) {
    const unsigned kc = clamp(k, nz - 1) - zb;
    v.x = at(ux, 8 * (sfx * kc + ox));
    v.y = at(uy, 8 * (sfy * kc + oy));
    v.yh = at(uy, 8 * (sfy * kc + oyh));
    v.zh = at(uz, 8 * (sxy * (clamp(k + 1, nz) - zb) + oc));
  };
  // class of a taken-up request for plane k (0 outside the box)
  auto cls_of = [&](int k, const Den& d) { return in && k >= 0 && k < nz ? (int)d.c : 0; };
  auto outer_of = [&](int k, const Den& d) { return ino && k >= 0 && k < nz && d.oc != 0 ? d.o : kNaN; };
  // planes k - 1, k, k + 1 of the own column at k = z0 - 1
  double nm, nc, np, no;
  int cc, cp;
  double vzl;   // low z face of plane k
  Vlow v0, v1;
  Den d0, d1;
  {
    Den a, b, c;
    load_n(z0 - 2, a);
    load_n(z0 - 1, b);
    load_n(z0, c);
    vzl = at(uz, 8 * (sxy * (clamp(z0 - 1, nz) - zb) + oc));
    load_u(z0 - 1, v0);
    load_n(z0 + 1, d0);
    load_u(z0, v1);
    load_n(z0 + 2, d1);
    cc = cls_of(z0 - 1, b);
    cp = cls_of(z0, c);
    nm = cls_of(z0 - 2, a) ? a.v : kNaN;
    nc = cc ? b.v : kNaN;
    np = cp ? c.v : kNaN;
    no = outer_of(z0, c);
    if (outer) ln[(z0 - 1) & 1][wo][lane] = outer_of(z0 - 1, b);
    ln[(z0 - 1) & 1][w + 1][lane] = nc;
  }
  __syncthreads();
  // what a plane leaves to the next one: z base, slope and gas, the low fluxes
  // and the density of the cell still open
  struct Open {
    double bz, sz, fxl, fxh, fyl, fzl, n;
    bool gas;
    int cls;
  };
  Open pr = {0, 0, 0, 0, 0, 0, 0, false, 0};
  // plane k: v holds its velocities, d the request for plane k + 2
  auto step = [&](int k, Vlow& v, Den& d) {
    const int pb = k & 1;
    const double vx0 = v.x, vy0 = v.y, vzh = v.zh;
    // slopes and bases at plane k
    const bool gas = cc != 0;
    const double yl = ln[pb][w][lane], yh = ln[pb][w + 2][lane];
    const double xl = lane_below(nc), xh = lane_above(nc);
    const double sx = adv_mc(nc - xl, xh - nc), sy = adv_mc(nc - yl, yh - nc), sz = adv_mc(nc - nm, np - nc);
    const double vx = 0.5 * (vx0 + lane_above(vx0)), vy = 0.5 * (vy0 + v.yh), vz = 0.5 * (vzl + vzh);
    // NaN in cells without gas, whose fluxes are not used
    const double bx = nc - c1 * (vy * sy + vz * sz);
    const double by = nc - c1 * (vx * sx + vz * sz);
    const double bz = nc - c1 * (vx * sx + vy * sy);
    const unsigned long long gm = __ballot(gas);
    lb[pb][w][lane] = by;
    ls[pb][w][lane] = sy;
    if (lane == 0) lg[pb][w] = gm;
    ln[pb ^ 1][w + 1][lane] = np;
    if (outer) ln[pb ^ 1][wo][lane] = no;
    load_u(k + 2, v);
    __syncthreads();
    // low-face fluxes of plane k
    auto face = [&](double u, bool g, double b, double s) {
      const double f = u * (b + (__builtin_copysign(0.5, u) - u * c2) * s);
      return g ? f : 0.0;
    };
    const int wd = max(w - 1, 0);
    const unsigned long long gdv = lg[pb][wd];   // uniform: a lane's bit through a scalar mask
    const unsigned long long gd =
        ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(gdv >> 32)) << 32) |
        (unsigned)__builtin_amdgcn_readfirstlane((int)gdv);
    const bool gxd = __builtin_amdgcn_inverse_ballot_w64(gm << 1), gyd = __builtin_amdgcn_inverse_ballot_w64(gd);
    const double byd = lb[pb][wd][lane], syd = ls[pb][wd][lane];
    const double bxd = lane_below(bx), sxd = lane_below(sx);
    const bool upx = vx0 >= 0.0, upy = vy0 >= 0.0, upz = vzl >= 0.0;
    double fx = face(vx0, upx ? gxd : gas, upx ? bxd : bx, upx ? sxd : sx);
    double fy = face(vy0, upy ? gyd : gas, upy ? byd : by, upy ? syd : sy);
    double fz = face(vzl, upz ? pr.gas : gas, upz ? pr.bz : bz, upz ? pr.sz : sz);
    if (edge) {   // inflow through the domain faces
      if (i == 0 && upx) fx = vx0 * inx0;
      if (i == nx && !upx) fx = vx0 * inx1;
      if (j == 0 && upy) fy = vy0 * iny0;
      if (j == ny && !upy) fy = vy0 * iny1;
    }
    if (k == 0 && upz) fz = vzl * inz0;
    if (k == nz && !upz) fz = vzl * inz1;
    lf[pb][w][lane] = fy;
    // close the cell of plane k - 1
    if (out && k > z0) {
      const double fyh = lf[pb ^ 1][w + 1][lane];
      const unsigned q = 8 * (sxy * (k - 1 - zb) + oc);
      if (pr.cls == 0) {
        at(nob, q) = 0.0;
      } else if (pr.cls != 2) {
        const double dc = ((pr.fxh - pr.fxl) + (fyh - pr.fyl) + (fz - pr.fzl)) * rh;
        if (pr.cls == 3) at(Dcb, q) = dc;
        at(nob, q) = pr.n - dt * dc;
      }
      if (pr.cls >= 2) {
        const unsigned qx = 8 * (sfx * (k - 1 - zb) + ox), qy = sfy * (k - 1 - zb);
        at(Fx, qx) = pr.fxl;
        at(Fx, qx + 8) = pr.fxh;
        at(Fy, 8 * (qy + oy)) = pr.fyl;
        at(Fy, 8 * (qy + oyh)) = fyh;
        at(Fz, q) = pr.fzl;
        at(Fz, q + 8 * sxy) = fz;
      }
    }
    pr = {bz, sz, fx, lane_above(fx), fy, fz, nc, gas, cc};
    cc = cp;
    cp = cls_of(k + 2, d);
    nm = nc;
    nc = np;
    np = cp ? d.v : kNaN;
    if (outer) no = outer_of(k + 2, d);
    load_n(k + 4, d);
    vzl = vzh;
  };
  for (int k = z0 - 1; k <= z1; k += 2) {
    step(k, v0, d0);
    if (k < z1) step(k + 1, v1, d1);
  }
}

}  // namespace ebmg
