// Plain Yee updates of one cell, shared by the plain passes (yee_plain.hip) and the
// workgroups of the fused sweep's launch that take the shell's H pass, and the soft sources,
// which ride in the scatter's launch.
#pragma once
#include <algorithm>

#include "mlk_internal.h"
#include "yee_common.h"

namespace mlk {

// H^{n+1/2} at cell (i,j,k) from E^n of `in`.
template <bool NT, typename T>
__device__ __forceinline__ void update_h_cell(const FieldPtrs<T>& in, const FieldPtrs<T>& out,
                                              const Geom& g, int i, int j, int k) {
  // products are not contracted into fused multiply-adds, as in the fused sweep,
  // so that every way of splitting the grid between the two rounds alike
#pragma clang fp contract(off)
  const size_t sx = 1, sy = (size_t)g.n[0], sz = (size_t)g.n[0] * g.n[1];
  const size_t id = cell_index(g, i, j, k);
  const T idx = (T)g.inv_dx;
  const T ex = in.E[0][id], ey = in.E[1][id], ez = in.E[2][id];
  T dEz_dy = (fwd(in.E[2], id, j, g.n[1], g.periodic[1], sy) - ez) * idx;
  T dEy_dz = (fwd(in.E[1], id, k, g.n[2], g.periodic[2], sz) - ey) * idx;
  T dEx_dz = (fwd(in.E[0], id, k, g.n[2], g.periodic[2], sz) - ex) * idx;
  T dEz_dx = (fwd(in.E[2], id, i, g.n[0], g.periodic[0], sx) - ez) * idx;
  T dEy_dx = (fwd(in.E[1], id, i, g.n[0], g.periodic[0], sx) - ey) * idx;
  T dEx_dy = (fwd(in.E[0], id, j, g.n[1], g.periodic[1], sy) - ex) * idx;
  const T o0 = in.H[0][id], o1 = in.H[1][id], o2 = in.H[2][id];
  const auto lx = layer_load(g, in.tab, in.psi, 1, 1, 2, 0, i, j, k);
  const auto ly = layer_load(g, in.tab, in.psi, 1, 0, 2, 1, i, j, k);
  const auto lz = layer_load(g, in.tab, in.psi, 1, 0, 1, 2, i, j, k);
  layer_apply(lx, out.psi, dEz_dx, dEy_dx);
  layer_apply(ly, out.psi, dEz_dy, dEx_dy);
  layer_apply(lz, out.psi, dEy_dz, dEx_dz);
  const T dt = (T)g.dt;
  const T h0 = o0 - dt * (dEz_dy - dEy_dz);
  const T h1 = o1 - dt * (dEx_dz - dEz_dx);
  const T h2 = o2 - dt * (dEy_dx - dEx_dy);
  store_field<NT>(&out.H[0][id], h0);
  store_field<NT>(&out.H[1][id], h1);
  store_field<NT>(&out.H[2][id], h2);
}

// E^{n+1} at cell (i,j,k); H^{n+1/2} is read from `out` (already advanced
// everywhere), E^n from `in`.
template <bool NT, typename T>
__device__ __forceinline__ void update_e_cell(const FieldPtrs<T>& in, const FieldPtrs<T>& out,
                                              const Geom& g, int i, int j, int k) {
  // products are not contracted into fused multiply-adds, as in the fused sweep,
  // so that every way of splitting the grid between the two rounds alike
#pragma clang fp contract(off)
  const size_t sx = 1, sy = (size_t)g.n[0], sz = (size_t)g.n[0] * g.n[1];
  const size_t id = cell_index(g, i, j, k);
  const T idx = (T)g.inv_dx;
  const T hx = out.H[0][id], hy = out.H[1][id], hz = out.H[2][id];
  T dHz_dy = (hz - bwd(out.H[2], id, j, g.n[1], g.periodic[1], sy)) * idx;
  T dHy_dz = (hy - bwd(out.H[1], id, k, g.n[2], g.periodic[2], sz)) * idx;
  T dHx_dz = (hx - bwd(out.H[0], id, k, g.n[2], g.periodic[2], sz)) * idx;
  T dHz_dx = (hz - bwd(out.H[2], id, i, g.n[0], g.periodic[0], sx)) * idx;
  T dHy_dx = (hy - bwd(out.H[1], id, i, g.n[0], g.periodic[0], sx)) * idx;
  T dHx_dy = (hx - bwd(out.H[0], id, j, g.n[1], g.periodic[1], sy)) * idx;
  const T ce = (T)g.dt * in.epsinv[id];
  const T e0 = in.E[0][id], e1 = in.E[1][id], e2 = in.E[2][id];
  const auto lx = layer_load(g, in.tab, in.psi, 0, 1, 2, 0, i, j, k);
  const auto ly = layer_load(g, in.tab, in.psi, 0, 0, 2, 1, i, j, k);
  const auto lz = layer_load(g, in.tab, in.psi, 0, 0, 1, 2, i, j, k);
  layer_apply(lx, out.psi, dHz_dx, dHy_dx);
  layer_apply(ly, out.psi, dHz_dy, dHx_dy);
  layer_apply(lz, out.psi, dHy_dz, dHx_dz);
  const T cx = dHz_dy - dHy_dz;
  const T cy = dHx_dz - dHz_dx;
  const T cz = dHy_dx - dHx_dy;
  const T n0 = tangential_wall(g, 0, i, j, k) ? T(0) : e0 + ce * cx;
  const T n1 = tangential_wall(g, 1, i, j, k) ? T(0) : e1 + ce * cy;
  const T n2 = tangential_wall(g, 2, i, j, k) ? T(0) : e2 + ce * cz;
  store_field<NT>(&out.E[0][id], n0);
  store_field<NT>(&out.E[1][id], n1);
  store_field<NT>(&out.E[2][id], n2);
}

// Whether cell (i,j,k) lies in the support of a source: its plane, or its one cell.
__device__ __forceinline__ bool source_covers(const Source& s, int i, int j, int k) {
  if (s.kind == 0) return (s.axis == 0 ? i : (s.axis == 1 ? j : k)) == s.index;
  return i == s.ijk[0] && j == s.ijk[1] && k == s.ijk[2];
}

// Soft source currents J at t = (n + 1/2) dt:  E -= (dt/eps_r) J.  One thread per
// cell of each source's support (a plane, or one cell); metallic-wall cells of
// the driven component keep E = 0.  Supports may share cells (two pulses on one plane, planes
// that cross, a point on a plane): the first source of a component on a cell adds those
// behind it there, in their order, so that a cell has one writer.
template <typename T>
__device__ __forceinline__ void source_body(const FieldPtrs<T>& f, const Geom& g,
                                            const SourceSet& src, int q, const StepNo& n, int t) {
  const Source& s = src.s[q];
  int i, j, k;
  if (s.kind == 0) {
    const int u = (s.axis + 1) % 3, v = (s.axis + 2) % 3;
    if (t >= g.n[u] * g.n[v]) return;
    int p[3];
    p[s.axis] = s.index;
    p[u] = t % g.n[u];
    p[v] = t / g.n[u];
    i = p[0];
    j = p[1];
    k = p[2];
  } else {
    if (t > 0) return;
    i = s.ijk[0];
    j = s.ijk[1];
    k = s.ijk[2];
  }
  if (tangential_wall(g, s.comp, i, j, k)) return;
  for (int o = 0; o < q; ++o)
    if (src.s[o].comp == s.comp && source_covers(src.s[o], i, j, k)) return;
  const double tm = ((double)n.get() + 0.5) * g.dt;
  const size_t id = cell_index(g, i, j, k);
  const double ei = f.epsinv ? (double)f.epsinv[id] : 1.0;  // null: eps_r = 1 everywhere
  T e = f.E[s.comp][id];
  for (int o = q; o < src.count; ++o) {
    const Source& so = src.s[o];
    if (so.comp != s.comp || !source_covers(so, i, j, k)) continue;
    const double scale = so.kind == 0 ? g.inv_dx : g.inv_dx * g.inv_dx * g.inv_dx;
    e -= (T)((double)g.dt * ei * (pulse_value(so, tm) * scale));
  }
  f.E[s.comp][id] = e;
}

// Blocks of 256 threads per source of a set (the largest support).
inline int source_blocks(const Geom& g, const SourceSet& src) {
  int maxp = 1;
  for (int q = 0; q < src.count; ++q)
    if (src.s[q].kind == 0) {
      const int u = (src.s[q].axis + 1) % 3, v = (src.s[q].axis + 2) % 3;
      maxp = std::max(maxp, g.n[u] * g.n[v]);
    }
  return (maxp + 255) / 256;
}

}  // namespace mlk
