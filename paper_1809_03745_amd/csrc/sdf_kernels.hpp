// Signed distance from a triangle mesh at the nodes of a box (the
// geometry-generation section of the paper: the distance to the closest
// polygon, edge or vertex, found through a bounding-volume hierarchy by a
// nearest-first closest-feature search): the search keeps the best squared
// distance found so far and descends into the nearer child box first, pushing
// the farther one while its box could still hold a closer triangle. The sign is
// that of (p - c) . n, with c the closest point and n the angle-weighted
// pseudonormal of the feature c lies on (face, edge or vertex), prepared on the
// host (mesh.cpp). FP64 throughout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ebmg {

constexpr int kSdfBlock = 256;
constexpr int kSdfStack = 48;   // pending subtrees per wavefront (at least the tree depth)

// oriented box of a tree node (MeshBox)
struct DevMeshBox {
  double ax[3][3], c[3], h[3];
  int32_t first, count;
};

// Closest point of triangle (a, b, c) to p by the Voronoi regions of its
// vertices, edges and face (the method of Ericson, Real-Time Collision
// Detection, section 5.1.5): returns the squared distance and the point,
// and the feature: 0 the face, 1 + j the edge from vertex j to j + 1 (mod 3),
// 4 + j vertex j.
__device__ __forceinline__ double closest_on_triangle(const double* __restrict__ r, double px, double py, double pz,
                                                      double& cx, double& cy, double& cz, int& feat) {
  const double ax = r[0], ay = r[1], az = r[2];
  const double bx = r[3], by = r[4], bz = r[5];
  const double qx = r[6], qy = r[7], qz = r[8];
  const double abx = bx - ax, aby = by - ay, abz = bz - az;
  const double acx = qx - ax, acy = qy - ay, acz = qz - az;
  const double apx = px - ax, apy = py - ay, apz = pz - az;
  const double d1 = abx * apx + aby * apy + abz * apz;
  const double d2 = acx * apx + acy * apy + acz * apz;
  if (d1 <= 0.0 && d2 <= 0.0) {
    cx = ax; cy = ay; cz = az;
    feat = 4;
  } else {
    const double bpx = px - bx, bpy = py - by, bpz = pz - bz;
    const double d3 = abx * bpx + aby * bpy + abz * bpz;
    const double d4 = acx * bpx + acy * bpy + acz * bpz;
    const double cpx = px - qx, cpy = py - qy, cpz = pz - qz;
    const double d5 = abx * cpx + aby * cpy + abz * cpz;
    const double d6 = acx * cpx + acy * cpy + acz * cpz;
    const double vc = d1 * d4 - d3 * d2;
    const double vb = d5 * d2 - d1 * d6;
    const double va = d3 * d6 - d5 * d4;
    if (d3 >= 0.0 && d4 <= d3) {
      cx = bx; cy = by; cz = bz;
      feat = 5;
    } else if (d6 >= 0.0 && d5 <= d6) {
      cx = qx; cy = qy; cz = qz;
      feat = 6;
    } else if (vc <= 0.0 && d1 >= 0.0 && d3 <= 0.0) {
      const double v = d1 / (d1 - d3);
      cx = ax + v * abx; cy = ay + v * aby; cz = az + v * abz;
      feat = 1;
    } else if (vb <= 0.0 && d2 >= 0.0 && d6 <= 0.0) {
      const double w = d2 / (d2 - d6);
      cx = ax + w * acx; cy = ay + w * acy; cz = az + w * acz;
      feat = 3;
    } else if (va <= 0.0 && (d4 - d3) >= 0.0 && (d5 - d6) >= 0.0) {
      const double w = (d4 - d3) / ((d4 - d3) + (d5 - d6));
      cx = bx + w * (qx - bx); cy = by + w * (qy - by); cz = bz + w * (qz - bz);
      feat = 2;
    } else {
      const double den = 1.0 / (va + vb + vc);
      const double v = vb * den, w = vc * den;
      cx = ax + abx * v + acx * w; cy = ay + aby * v + acy * w; cz = az + abz * v + acz * w;
      feat = 0;
    }
  }
  const double dx = px - cx, dy = py - cy, dz = pz - cz;
  return dx * dx + dy * dy + dz * dz;
}

__device__ __forceinline__ double box_d2(const DevMeshBox& n, double px, double py, double pz) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double t = n.ax[k][0] * px + n.ax[k][1] * py + n.ax[k][2] * pz - n.c[k];
    const double e = fmax(fabs(t) - n.h[k], 0.0);
    s += e * e;
  }
  return s;
}

// What the search reads of a triangle: the smallest disc around it (unit
// normal, centre, radius), and vertex a, the edges ab and ac and their
// products ab.ab, ab.ac, ac.ac.
struct DevDisc {
  double n[3], c[3], rad, pad;
};
struct DevSearchTri {
  double a[3], ab[3], ac[3], bb, bc, cc;
};

// A lower bound of the squared distance to the disc: the height above its
// plane and the part of the lateral offset beyond its radius (a little less,
// for the rounding of the difference and of the approximate root).
__device__ __forceinline__ double disc_d2(const DevDisc& t, double px, double py, double pz) {
  const double x = px - t.c[0], y = py - t.c[1], z = pz - t.c[2];
  const double hh = t.n[0] * x + t.n[1] * y + t.n[2] * z;
  const double lat2 = fmax((x * x + y * y + z * z) * (1.0 - 1e-14) - hh * hh, 1e-300);
  const double l = fmax(lat2 * __builtin_amdgcn_rsq(lat2) * (1.0 - 1e-6) - t.rad, 0.0);
  return hh * hh + l * l;
}

// Squared distance of p to a triangle in the regions of closest_on_triangle,
// with the products at b and c taken from those at a and one reciprocal. Only
// ranks the triangles: the closest point minimises the distance, so an error
// of its parameters enters squared.
__device__ __forceinline__ double search_d2(const DevSearchTri& t, double px, double py, double pz) {
  const double x = px - t.a[0], y = py - t.a[1], z = pz - t.a[2];
  const double d1 = t.ab[0] * x + t.ab[1] * y + t.ab[2] * z;
  const double d2 = t.ac[0] * x + t.ac[1] * y + t.ac[2] * z;
  const double d3 = d1 - t.bb, d4 = d2 - t.bc, d5 = d1 - t.bc, d6 = d2 - t.cc;
  const double vc = d1 * d4 - d3 * d2, vb = d5 * d2 - d1 * d6, va = d3 * d6 - d5 * d4;
  const double e1 = d4 - d3, e2 = d5 - d6;
  const bool ra = d1 <= 0.0 && d2 <= 0.0, rb = d3 >= 0.0 && d4 <= d3, rc = d6 >= 0.0 && d5 <= d6;
  const bool eab = vc <= 0.0 && d1 >= 0.0 && d3 <= 0.0, eac = vb <= 0.0 && d2 >= 0.0 && d6 <= 0.0;
  const bool ebc = va <= 0.0 && e1 >= 0.0 && e2 >= 0.0;
  // (v, w) = (nv, nw) / den; in edge order, so the first region that holds wins
  double nv = vb, nw = vc, den = va + vb + vc;
  if (ebc) { nv = e2; nw = e1; den = e1 + e2; }
  if (eac) { nv = 0.0; nw = d2; den = d2 - d6; }
  if (eab) { nv = d1; nw = 0.0; den = d1 - d3; }
  if (rc) { nv = 0.0; nw = 1.0; den = 1.0; }
  if (rb) { nv = 1.0; nw = 0.0; den = 1.0; }
  if (ra) { nv = 0.0; nw = 0.0; den = 1.0; }
  double q = __builtin_amdgcn_rcp(den);
  q = q * (2.0 - den * q);
  const double v = nv * q, w = nw * q;
  const double rx = x - v * t.ab[0] - w * t.ac[0], ry = y - v * t.ab[1] - w * t.ac[1],
               rz = z - v * t.ab[2] - w * t.ac[2];
  return rx * rx + ry * ry + rz * rz;
}

// sdf[node] for the nodes lo + (i, j, k) h of an (n0+1) x (n1+1) x (n2+1)
// lattice (x fastest); visits (nullable) accumulates the boxes and triangles
// that a node's own distance bound made the search examine.
//
// A wavefront searches for a brick of BX x BY x BZ nodes together:
// neighbouring nodes need nearly the same subtrees (1.1 to 1.5 times one
// node's for 4 x 4 x 4), so the walk is uniform: boxes and triangles come
// through scalar loads, siblings in one, and no lane waits for another's
// branch. A subtree is entered while any lane's best distance exceeds its box
// distance, nearer child first by vote, and a triangle is evaluated only if
// its disc is closer than some lane's best. The distance and the sign come
// from closest_on_triangle on the winner, the distance from the search itself
// where that found a clearly smaller one (slivers: evaluating every triangle
// and taking the least, as the search of one node does, never exceeded the
// distance to the nearest edge; the winner alone did, by up to 8e-6 on a
// unit-length prism 1e-6 wide). Bound by the FP64 arithmetic of the
// tests on large lattices, by the chain of loads along the walk on small ones.
// One thread per node with a stack and axis-aligned boxes took 4.1 ms for
// 129^3 nodes of a 6144-triangle pin and 28 ms at 257^3, its lanes diverging
// at every step; this form takes 0.83 and 4.0 ms (a third of the time saved by
// the oriented boxes and discs, which cut the tests per node from 257 to 97).
template <int BX, int BY, int BZ>
__global__ void __launch_bounds__(kSdfBlock) k_sdf_mesh(const DevMeshBox* __restrict__ boxes,
                                                       const DevDisc* __restrict__ disc,
                                                       const DevSearchTri* __restrict__ stri,
                                                       const double* __restrict__ tri, int m0, int m1, int m2,
                                                       double h, double lox, double loy, double loz,
                                                       double* __restrict__ sdf,
                                                       unsigned long long* __restrict__ visits) {
  constexpr double kSlack = 1.0 + 1e-12;   // for the rounding of the bounds
  __shared__ int32_t stk[kSdfBlock / 64][kSdfStack];
  __shared__ unsigned long long vsum[kSdfBlock / 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int b0 = (m0 + BX - 1) / BX, b1 = (m1 + BY - 1) / BY, b2 = (m2 + BZ - 1) / BZ;
  const int64_t brick = (int64_t)blockIdx.x * (kSdfBlock / 64) + wave;
  unsigned long long nvis = 0;
  if (brick < (int64_t)b0 * b1 * b2) {
    const int i = (int)(brick % b0) * BX + lane % BX;
    const int j = (int)((brick / b0) % b1) * BY + (lane / BX) % BY;
    const int k = (int)(brick / ((int64_t)b0 * b1)) * BZ + lane / (BX * BY);
    const bool in = lane < BX * BY * BZ && i < m0 && j < m1 && k < m2;
    const int nin = __popcll(__ballot(in));
    const double px = lox + i * h, py = loy + j * h, pz = loz + k * h;
    double best = in ? 1e300 : -1.0;   // squared distance so far; lanes without a node need nothing
    int win = -1;
    int sp = 0;
    int first = boxes[0].first, count = boxes[0].count;
    while (true) {
      bool down = false;
      if (count >= 0) {
        for (int t = first; t < first + count; ++t) {
          const unsigned long long need = __ballot(disc_d2(disc[t], px, py, pz) < best * kSlack);
          if (need == 0) continue;
          nvis += __popcll(need);
          const double d2 = search_d2(stri[t], px, py, pz);
          if (d2 < best) {
            best = d2;
            win = t;
          }
        }
      } else {
        const DevMeshBox* c = boxes - count;
        const DevMeshBox l = c[0], r = c[1];
        const double dl = box_d2(l, px, py, pz), dr = box_d2(r, px, py, pz);
        const unsigned long long nl = __ballot(dl < best * kSlack), nr = __ballot(dr < best * kSlack);
        nvis += __popcll(nl) + __popcll(nr);
        const bool lfirst = nr == 0 || (nl != 0 && 2 * __popcll(__ballot(in && dl <= dr)) >= nin);
        if (nl != 0 && nr != 0 && sp < kSdfStack) {
          stk[wave][sp] = lfirst ? 1 - count : -count;
          ++sp;
        }
        down = (nl | nr) != 0;
        first = lfirst ? l.first : r.first;
        count = lfirst ? l.count : r.count;
      }
      // next pending subtree that may still hold a closer triangle
      while (!down && sp > 0) {
        --sp;
        const DevMeshBox c = boxes[__builtin_amdgcn_readfirstlane(stk[wave][sp])];
        down = __ballot(box_d2(c, px, py, pz) < best * kSlack) != 0;
        first = c.first;
        count = c.count;
      }
      if (!down) break;
    }
    if (in) {
      double d = 1e150, side = 1.0;
      if (win >= 0) {
        const double* r = tri + (int64_t)win * 30;
        double cx, cy, cz;
        int f;
        // on a sliver either evaluation may place the closest point far along
        // its length; the smaller distance is the better one (elsewhere they
        // agree to rounding, and the first is kept)
        const double d2 = closest_on_triangle(r, px, py, pz, cx, cy, cz, f);
        d = sqrt(best < d2 * (1.0 - 1e-9) ? best : d2);
        const double* nrm = f == 0 ? r + 9 : (f <= 3 ? r + 12 + 3 * (f - 1) : r + 21 + 3 * (f - 4));
        side = (px - cx) * nrm[0] + (py - cy) * nrm[1] + (pz - cz) * nrm[2];
      }
      sdf[i + (int64_t)m0 * (j + (int64_t)m1 * k)] = side >= 0.0 ? d : -d;
    }
  }
  if (visits) {
    // per-wavefront sums, then one atomic per block
    if (lane == 0) vsum[wave] = nvis;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long s = 0;
      for (int w = 0; w < kSdfBlock / 64; ++w) s += vsum[w];
      atomicAdd(visits, s);
    }
  }
}

}  // namespace ebmg
