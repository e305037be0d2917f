// Multigrid hierarchy: coarse levels, transfer lists, colouring, bottom inverse.
//
// The paper's solver is the residual-correction geometric multigrid of its
// multigrid-solver subsection; the coarse operators are not specified there
// (EBChombo coarsens the EB graph). Here each coarse cell aggregates 2^D fine
// cells and carries one unknown per phase present among its children. Rows of
// coarse cells whose children are all regular cells of one phase (and whose
// neighbours share that primary phase) are the rediscretised (2D+1)-point
// template at spacing 2h; every other coarse row is the Galerkin product of the
// fine rows with piecewise-constant prolongation, its flux part scaled by
// 2^-(D+1) and its mass part by 2^-D, which equals the rediscretised template
// wherever both apply. Odd extents coarsen too, to (n + 1) / 2 cells (the last
// over one fine cell). Restriction averages the 2^D children (covered children
// count as zero residual), prolongation injects. Only the convergence rate
// depends on these choices; the fixed point is the finest-level system.
#include <algorithm>
#include <cmath>
#include <unordered_map>

#include "internal.hpp"

namespace ebmg {

namespace {

inline void cell_ijk(const Grid& g, int64_t c, int* ijk) {
  ijk[0] = (int)(c % g.n[0]);
  ijk[1] = (int)((c / g.n[0]) % g.n[1]);
  ijk[2] = (int)(c / ((int64_t)g.n[0] * g.n[1]));
}

std::vector<int32_t> irow_index(const Level& L) {
  std::vector<int32_t> m(L.N + L.N2, -1);
  for (size_t r = 0; r < L.irow_dof.size(); ++r) m[L.irow_dof[r]] = (int32_t)r;
  return m;
}

}  // namespace

// d(flux)/d(cell value) of domain face f's closure for a cell of width w
// along the face's axis and coefficient b.
static double wall_slope(const Problem& pb, int f, double b, double w) {
  const int kind = pb.bc.kind[f];
  if (kind == EBMG_BC_NEUMANN) return 0.0;
  if (kind == EBMG_BC_DIRICHLET) return -2.0 * b / w;
  const double a1 = pb.bc.robin_a1[f], a2 = pb.bc.robin_a2[f];
  return -(b * a1 / a2) / (1.0 + 0.5 * w * a1 / a2);
}

// Rediscretised template constants of a coarse level at its own spacing.
void coarse_template(Level& C, const Problem& pb) {
  const double h = C.g.h, beta = pb.opt.beta;
  for (int p = 0; p < 2; ++p) {
    const double b = pb.bph[p];
    C.coff[p] = beta * b / (h * h);
    C.mass[p] = pb.opt.alpha * pb.aph[p];
    C.d0[p] = C.mass[p] - 2.0 * C.g.dim * C.coff[p];
    for (int f = 0; f < 2 * C.g.dim; ++f) {
      C.cb[f][p] = (beta / h) * wall_slope(pb, f, b, h) + C.coff[p];
    }
  }
}


void Level::row(int64_t q, double& mass_out, std::vector<std::pair<int64_t, double>>& out) const {
  out.clear();
  mass_out = 0;
  int64_t cell = q < N ? q : sec_cell[q - N];
  uint8_t t = tag[cell] & 3;
  if (q < N && t <= 1) {
    int c[3];
    cell_ijk(g, cell, c);
    double dg = d0[t];
    for (int d = 0; d < g.dim; ++d)
      for (int side = 0; side < 2; ++side) {
        int nb[3] = {c[0], c[1], c[2]};
        nb[d] += side ? 1 : -1;
        if (nb[d] >= 0 && nb[d] < g.n[d])
          out.emplace_back(g.cell(nb[0], nb[1], nb[2]), coff[t]);
        else
          dg += cb[2 * d + side][t];
      }
    mass_out = mass[t];
    out.emplace_back(q, dg - mass[t]);
    return;
  }
  if (t == TAG_COV && q < N) return;
  // irregular: linear search is avoided by the caller's index when available
  auto it = std::lower_bound(irow_dof.begin(), irow_dof.end(), q);
  if (it == irow_dof.end() || *it != q) throw std::logic_error("missing irregular row");
  size_t r = it - irow_dof.begin();
  mass_out = imass[r];
  out.emplace_back(q, idiag[r] - imass[r]);
  for (int64_t e = rp[r]; e < rp[r + 1]; ++e) out.emplace_back(col[e], val[e]);
}

// Explicit rows grouped by the red/black colour of their cell (group 0: red,
// i+j+k even), in row order within a group.
void colour_irregular(Level& L) {
  const size_t R = L.irow_dof.size();
  L.cls_ptr.assign(3, 0);
  L.cls_rows.clear();
  L.cls_rows.reserve(R);
  for (int grp = 0; grp < 2; ++grp) {
    for (size_t r = 0; r < R; ++r) {
      const int64_t q = L.irow_dof[r];
      const int64_t cell = q < L.N ? q : L.sec_cell[q - L.N];
      int ijk[3];
      cell_ijk(L.g, cell, ijk);
      if (((ijk[0] + ijk[1] + ijk[2]) & 1) == grp) L.cls_rows.push_back((int32_t)r);
    }
    L.cls_ptr[grp + 1] = (int32_t)L.cls_rows.size();
  }
}

namespace {

// The aggregation of a level's cells: a coarse cell holds the 2^D fine cells
// at twice its index, fewer at the high end of an axis of odd extent.
struct Agg {
  const Level& L;
  const Level& C;
  int64_t parent(int64_t c) const {
    int ijk[3];
    cell_ijk(L.g, c, ijk);
    return C.g.cell(ijk[0] / 2, ijk[1] / 2, L.g.dim == 3 ? ijk[2] / 2 : 0);
  }
  // child q of coarse cell P, -1 past the end of an odd axis
  int64_t child(int64_t P, int q) const {
    int ijk[3];
    cell_ijk(C.g, P, ijk);
    const int i = 2 * ijk[0] + (q & 1), j = 2 * ijk[1] + ((q >> 1) & 1);
    const int k = L.g.dim == 3 ? 2 * ijk[2] + ((q >> 2) & 1) : 0;
    if (i >= L.g.n[0] || j >= L.g.n[1] || (L.g.dim == 3 && k >= L.g.n[2])) return -1;
    return L.g.cell(i, j, k);
  }
  int64_t cdof(int64_t P, int p) const { return C.primary[P] == p ? P : C.N + C.sec_of[P]; }
  // the coarse unknown that holds fine unknown q
  int64_t agg(int64_t q) const {
    return cdof(parent(q < L.N ? q : L.sec_cell[q - L.N]), q < L.N ? L.primary[q] : 1);
  }
};

}  // namespace

// Whether cell P's template would reach a last cell that lies partly outside
// the box (under an odd extent), as its own or as a neighbour.
static bool near_partial(const Level& C, const int* ijk) {
  for (int d = 0; d < C.g.dim; ++d)
    if (C.fill[d] < 1.0 && ijk[d] >= C.g.n[d] - 2) return true;
  return false;
}

// Row of a pure cell near a partly filled last cell: the finite-volume row on
// the tensor grid whose last cells have their true widths (in units of the
// level's spacing), scaled like the template rows. With the plain Galerkin
// product there the distance to the wall is off by up to two per level, and a
// 250^2 Dirichlet box took over 100 V-cycles to 1e-10 where it takes 14 (256^2: 11).
static void partial_row(const Problem& pb, const Level& C, int64_t P, double& mass, double& dg,
                        std::vector<std::pair<int64_t, double>>& ent) {
  int ijk[3];
  cell_ijk(C.g, P, ijk);
  const int D = C.g.dim, p = C.primary[P];
  const double h = C.g.h;
  auto width = [&](int d, int i) { return i == C.g.n[d] - 1 ? C.fill[d] : 1.0; };
  double vol = 1.0;
  for (int d = 0; d < D; ++d) vol *= width(d, ijk[d]);
  mass = C.mass[p] * vol;
  dg = mass;
  ent.clear();
  for (int d = 0; d < D; ++d) {
    const double w = width(d, ijk[d]), area = vol / w;
    for (int side = 0; side < 2; ++side) {
      int nb[3] = {ijk[0], ijk[1], ijk[2]};
      nb[d] += side ? 1 : -1;
      if (nb[d] >= 0 && nb[d] < C.g.n[d]) {
        const double v = C.coff[p] * area / (0.5 * (w + width(d, nb[d])));
        ent.emplace_back(C.g.cell(nb[0], nb[1], nb[2]), v);
        dg -= v;
      } else {
        dg += (pb.opt.beta / h) * wall_slope(pb, 2 * d + side, pb.bph[p], w * h) * area;
      }
    }
  }
}

// The explicit coarse rows (primaries of irregular cells in cell order, then
// secondaries): partial_row where it applies, else the Galerkin products of
// the fine rows. Fills C's row arrays; on a hierarchy whose coefficients
// changed it gives the same rows and columns with new values.
void coarse_rows(const Problem& pb, const Level& L, Level& C) {
  const Agg G{L, C};
  const int nch = 1 << L.g.dim;
  const double sflux = 1.0 / (double)(2 * nch), smass = 1.0 / (double)nch;
  std::vector<std::pair<int64_t, double>> rowbuf, ent;
  std::unordered_map<int64_t, double> acc;
  std::vector<int64_t> todo;
  for (int64_t P = 0; P < C.N; ++P)
    if ((C.tag[P] & 3) == TAG_IRR) todo.push_back(P);
  for (int64_t s = 0; s < C.N2; ++s) todo.push_back(C.N + s);
  C.rp.assign(1, 0);
  C.col.clear();
  C.val.clear();
  C.irow_dof.clear();
  C.idiag.clear();
  C.imass.clear();
  for (int64_t J : todo) {
    const int64_t P = J < C.N ? J : C.sec_cell[J - C.N];
    const int pj = J < C.N ? C.primary[P] : 1;
    acc.clear();
    double mass = 0, dg = 0;
    const bool part = J < C.N && C.pure[P];
    if (part) partial_row(pb, C, P, mass, dg, ent);
    for (int q = 0; q < nch && !part; ++q) {
      const int64_t c = G.child(P, q);
      if (c < 0) continue;
      int64_t fd[2];
      int nf = 0;
      if (L.primary[c] == pj) fd[nf++] = c;
      if (pj == 1 && L.sec_of[c] >= 0) fd[nf++] = L.N + L.sec_of[c];
      for (int t = 0; t < nf; ++t) {
        double m;
        L.row(fd[t], m, rowbuf);
        mass += smass * m;
        for (auto& e : rowbuf) acc[G.agg(e.first)] += sflux * e.second;
      }
    }
    if (!part) {
      dg = mass;
      ent.clear();
      for (auto& kv : acc) {
        if (kv.first == J)
          dg += kv.second;
        else
          ent.emplace_back(kv.first, kv.second);
      }
    }
    std::sort(ent.begin(), ent.end());
    for (auto& e : ent) {
      C.col.push_back((int32_t)e.first);
      C.val.push_back(e.second);
    }
    C.irow_dof.push_back(J);
    C.idiag.push_back(dg);
    C.imass.push_back(mass);
    C.rp.push_back((int64_t)C.col.size());
  }
}

// One coarsening. An axis of odd extent gets (n + 1) / 2 coarse cells, the
// last of them over one fine cell; the cells there carry explicit rows, and
// those with missing children are restricted and prolonged by list. Stopping
// at the first odd extent instead left bottom levels of thousands of
// unknowns (a 1000^2 box ends at 125^2), whose solve was all but 5 ms of a
// 0.98 s solve there and 0.32 of 0.33 s at 100^3. A first odd level that the
// dense inverse can still take is the bottom: its product costs less than the
// further levels' launches, and the cycle solves it exactly (488^2 two disks
// ending at 61^2 instead of 16^2: 2.76 -> 2.23 ms, 72^3 pin 4.81 -> 4.06 ms).
// That is the rule for solves and set-ups; a box that takes new coefficients
// also pays for the larger inverse each time (12 ms at 61^2, 1.3 ms at 33^2).
static bool coarsen(Problem& pb, size_t lf) {
  Level& L = pb.levels[lf];
  const Grid& gf = L.g;
  bool odd = false, even_so_far = true;
  for (int d = 0; d < gf.dim; ++d) {
    if (gf.n[d] < 4) return false;
    odd = odd || gf.n[d] % 2;
    even_so_far = even_so_far && L.fill[d] == 1.0;
  }
  if (odd && even_so_far && L.ndof() <= kBottomMax) return false;
  Level C;
  C.g = gf;
  for (int d = 0; d < gf.dim; ++d) {
    C.g.n[d] = (gf.n[d] + 1) / 2;
    C.fill[d] = gf.n[d] % 2 ? 0.5 * L.fill[d] : 0.5 * (1.0 + L.fill[d]);
  }
  C.g.h = 2 * gf.h;
  const Grid& gc = C.g;
  const int D = gf.dim;
  const int nch = 1 << D;
  C.N = gc.ncell();
  const Agg G{L, C};
  std::vector<uint8_t> has(C.N, 0);
  for (int64_t c = 0; c < L.N; ++c) {
    int64_t P = G.parent(c);
    if (L.primary[c] == 0) has[P] |= 1;
    if (L.primary[c] == 1) has[P] |= 2;
    if (L.sec_of[c] >= 0) has[P] |= 2;
  }
  C.primary.assign(C.N, -1);
  C.sec_of.assign(C.N, -1);
  for (int64_t P = 0; P < C.N; ++P) {
    C.primary[P] = (has[P] & 1) ? 0 : ((has[P] & 2) ? 1 : -1);
    if (has[P] == 3) {
      C.sec_of[P] = (int32_t)C.sec_cell.size();
      C.sec_cell.push_back((int32_t)P);
    }
  }
  C.N2 = (int64_t)C.sec_cell.size();
  auto fine_cell = [&](int64_t q) -> int64_t { return q < L.N ? q : L.sec_cell[q - L.N]; };
  // tags
  C.tag.assign(C.N, TAG_IRR);
  C.pure.assign(C.N, 0);
  std::vector<uint8_t> simple(C.N, 1);
  for (int64_t P = 0; P < C.N; ++P) {
    int pc = C.primary[P];
    if (pc < 0) {
      C.tag[P] = TAG_COV;
      continue;
    }
    bool allreg = true;
    for (int q = 0; q < nch; ++q) {
      int64_t c = G.child(P, q);
      if (c < 0) {
        simple[P] = 0;
        continue;
      }
      if (L.sec_of[c] >= 0 || (L.primary[c] >= 0 && L.primary[c] != pc)) simple[P] = 0;
      if (L.pure.empty() ? (L.tag[c] & 3) != pc : !(L.pure[c] && L.primary[c] == pc)) allreg = false;
    }
    int ijk[3];
    cell_ijk(gc, P, ijk);
    if (allreg) {
      for (int d = 0; d < D && allreg; ++d)
        for (int side = 0; side < 2; ++side) {
          int nb[3] = {ijk[0], ijk[1], ijk[2]};
          nb[d] += side ? 1 : -1;
          if (nb[d] >= 0 && nb[d] < gc.n[d] && C.primary[gc.cell(nb[0], nb[1], nb[2])] != pc) allreg = false;
        }
    }
    C.pure[P] = allreg;
    C.tag[P] = allreg && !near_partial(C, ijk) ? (uint8_t)pc : (uint8_t)TAG_IRR;
    if (!simple[P]) C.tag[P] |= TAG_NONSIMPLE;
  }
  coarse_template(C, pb);
  coarse_rows(pb, L, C);
  // transfer lists for non-simple coarse cells
  L.ns_cdof.clear();
  L.ns_ptr.assign(1, 0);
  L.ns_child.clear();
  L.np_fdof.clear();
  L.np_cdof.clear();
  for (int64_t P = 0; P < C.N; ++P) {
    if (simple[P] || C.primary[P] < 0) continue;
    for (int ph = 0; ph < 2; ++ph) {
      if (!((has[P] >> ph) & 1)) continue;
      const int64_t J = G.cdof(P, ph);
      L.ns_cdof.push_back(J);
      for (int q = 0; q < nch; ++q) {
        int64_t c = G.child(P, q);
        if (c < 0) continue;
        if (L.primary[c] == ph) L.ns_child.push_back(c);
        if (ph == 1 && L.sec_of[c] >= 0) L.ns_child.push_back(L.N + L.sec_of[c]);
      }
      L.ns_ptr.push_back((int32_t)L.ns_child.size());
    }
  }
  for (int64_t q = 0; q < L.N + L.N2; ++q) {
    int64_t c = fine_cell(q);
    if (q < L.N && L.primary[c] < 0) continue;
    int64_t P = G.parent(c);
    if (simple[P]) continue;
    L.np_fdof.push_back(q);
    L.np_cdof.push_back(G.agg(q));
  }
  colour_irregular(C);
  pb.levels.push_back(std::move(C));
  return true;
}

static void dense_inverse(std::vector<double>& A, int64_t n) {
  std::vector<double> I(n * n, 0.0);
  for (int64_t i = 0; i < n; ++i) I[i * n + i] = 1.0;
  for (int64_t c = 0; c < n; ++c) {
    int64_t piv = c;
    double best = std::fabs(A[c * n + c]);
    for (int64_t r = c + 1; r < n; ++r)
      if (std::fabs(A[r * n + c]) > best) {
        best = std::fabs(A[r * n + c]);
        piv = r;
      }
    if (best == 0.0) throw GeomError("singular bottom-level operator");
    if (piv != c)
      for (int64_t k = 0; k < n; ++k) {
        std::swap(A[c * n + k], A[piv * n + k]);
        std::swap(I[c * n + k], I[piv * n + k]);
      }
    const double inv = 1.0 / A[c * n + c];
    for (int64_t k = 0; k < n; ++k) {
      A[c * n + k] *= inv;
      I[c * n + k] *= inv;
    }
    for (int64_t r = 0; r < n; ++r) {
      if (r == c) continue;
      const double f = A[r * n + c];
      if (f == 0.0) continue;
      for (int64_t k = 0; k < n; ++k) {
        A[r * n + k] -= f * A[c * n + k];
        I[r * n + k] -= f * I[c * n + k];
      }
    }
  }
  A.swap(I);
}

void build_hierarchy(Problem& pb) {
  colour_irregular(pb.levels[0]);
  while (pb.levels.size() < 16 && pb.levels.back().ndof() > pb.opt.bottom_max) {
    if (!coarsen(pb, pb.levels.size() - 1)) break;
  }
  build_bottom(pb);
}

// Dense FP64 inverse of the coarsest level (left empty above kBottomMax
// unknowns, where the bottom is solved by Krylov iterations, and where the
// device forms it).
void build_bottom(Problem& pb) {
  const Level& B = pb.levels.back();
  const int64_t n = B.ndof();
  pb.bottom_n = n;
  pb.bottom_inv.clear();
  if (n > kBottomMax || !pb.host_bottom) return;
  std::vector<double> A(n * n, 0.0);
  std::vector<std::pair<int64_t, double>> rowbuf;
  for (int64_t q = 0; q < n; ++q) {
    int64_t cell = q < B.N ? q : B.sec_cell[q - B.N];
    if (q < B.N && B.primary[cell] < 0) {
      A[q * n + q] = 1.0;
      continue;
    }
    double m;
    B.row(q, m, rowbuf);
    A[q * n + q] += m;
    for (auto& e : rowbuf) A[q * n + e.first] += e.second;
  }
  dense_inverse(A, n);
  pb.bottom_inv.swap(A);
}

}  // namespace ebmg
