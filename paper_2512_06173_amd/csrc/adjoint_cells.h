// Cell updates of the transposed step (see adjoint.hip), shared by its passes and by the
// workgroups of the fused transposed sweep's launch that take the E pass of the shell.
#pragma once
#include "mlk_internal.h"
#include "yee_common.h"

namespace mlk {

template <typename T>
struct AdjPtrs {
  T* E[3];           // adjoint of E
  T* H[3];           // adjoint of H
  const T* epsinv;   // null in vacuum (eps_r = 1) for the transposed sweep
  const T* tab;      // CPML tables (b, c, 1/kappa) of the forward sweep
  const T* psi_in;   // adjoint of psi (both fields), read
  T* psi_out;        // adjoint of psi, written
};

// Adjoint of the plain derivative of component c along the axis of l from w, the adjoint of
// the stretched one (l.p0 and l.p1 belong to the axis's lower and higher other component).
template <typename T>
__device__ __forceinline__ T dbar(const LayerTerm<T>& l, bool first, T w) {
  return l.on ? (l.ik + l.c) * w + l.c * (first ? l.p0 : l.p1) : w;
}

template <typename T>
__device__ __forceinline__ void psib_update(const LayerTerm<T>& l, bool first, T* psi_out, T w) {
  if (l.on) psi_out[first ? l.o0 : l.o1] = l.b * (w + (first ? l.p0 : l.p1));
}

// The two components other than axis a, and whether c is the lower of them.
__device__ __forceinline__ constexpr int other0(int a) { return a == 0 ? 1 : 0; }
__device__ __forceinline__ constexpr int other1(int a) { return a == 2 ? 1 : 2; }

// A cell's neighbour one step along each axis (dir = +1 or -1): linear index,
// coordinate along the axis, existence (false beyond a non-periodic face) and
// CPML-layer membership.
struct Nbrs {
  size_t id[3];
  int q[3];
  bool ok[3], lay[3];
};

__device__ __forceinline__ Nbrs neighbours(const Geom& g, int i, int j, int k, size_t id, int dir) {
  const size_t st[3] = {1, (size_t)g.n[0], (size_t)g.n[0] * g.n[1]};
  const int q0[3] = {i, j, k};
  Nbrs nb;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int q = q0[a] + dir;
    size_t nid = dir > 0 ? id + st[a] : id - st[a];
    bool ok = true;
    if (q < 0 || q >= g.n[a]) {
      ok = g.periodic[a] != 0;
      q = q < 0 ? q + g.n[a] : q - g.n[a];
      nid = dir > 0 ? id - (size_t)(g.n[a] - 1) * st[a] : id + (size_t)(g.n[a] - 1) * st[a];
    }
    nb.id[a] = ok ? nid : id;
    nb.q[a] = q;
    nb.ok[a] = ok;
    nb.lay[a] = ok && has_cpml(g, a) && in_layer(g, a, q);
  }
  return nb;
}

// curl terms of component c: derivative axis and component of the other field,
// with the sign of the term
constexpr int kAx[3][2] = {{1, 2}, {2, 0}, {0, 1}};
constexpr int kOt[3][2] = {{2, 1}, {0, 2}, {1, 0}};

// The psi adjoint and coefficients of a cell's and its neighbours' derivatives of `field`,
// per axis.
template <typename T>
__device__ __forceinline__ void layers_load(const Geom& g, const AdjPtrs<T>& p, int field, int i,
                                            int j, int k, const Nbrs& nb, LayerTerm<T> (&own)[3],
                                            LayerTerm<T> (&nbr)[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    own[a] = layer_load(g, p.tab, p.psi_in, field, other0(a), other1(a), a, i, j, k);
    nbr[a] = LayerTerm<T>{};
    if (nb.lay[a])
      nbr[a] = layer_load(g, p.tab, p.psi_in, field, other0(a), other1(a), a,
                          a == 0 ? nb.q[0] : i, a == 1 ? nb.q[1] : j, a == 2 ? nb.q[2] : k);
  }
}

// Cell updates of the transposed step.  Every field load of a thread is issued
// up front, unconditionally (a missing neighbour reads the cell itself and its
// term is zeroed afterwards), and those of the CPML terms after them, so the loads are
// in flight together.  In place (OOP = false), p holds Eb and Hb;
// out of place, Eb and Hb are read from p and written to o.

// Transposed E update.  Eb holds the adjoint of E^{n+1}; Hb gains the curl
// part.  In place, Eb leaves holding that of E^n (identity part, zero on the
// walls, stored only where a wall zeroes it); out of place the H pass applies
// the mask.
template <typename T, bool OOP, bool NT>
__device__ __forceinline__ void adj_e_cell(const AdjPtrs<T>& p, const AdjPtrs<T>& o,
                                           const Geom& g, int i, int j, int k) {
  const size_t id = (size_t)i + (size_t)g.n[0] * ((size_t)j + (size_t)g.n[1] * (size_t)k);
  const T dt = (T)g.dt, idx = (T)g.inv_dx;
  const Nbrs nb = neighbours(g, i, j, k, id, +1);
  T eo[3], hv[3], en[3][3], epn[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) eo[c] = p.E[c][id];
  const T ei = p.epsinv ? p.epsinv[id] : T(1);  // null: eps_r = 1 everywhere
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    epn[a] = p.epsinv ? p.epsinv[nb.id[a]] : T(1);
#pragma unroll
    for (int c = 0; c < 3; ++c) en[a][c] = c != a ? p.E[c][nb.id[a]] : T(0);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) hv[c] = p.H[c][id];
  LayerTerm<T> own[3], nbr[3];
  layers_load(g, p, 0, i, j, k, nb, own, nbr);
  // wall planes through this cell (a wall zeroes the tangential E on it)
  const bool w0 = g.wall[0] && i == 0, w1 = g.wall[1] && j == 0, w2 = g.wall[2] && k == 0;
  const bool wl[3] = {w0, w1, w2};
  T u[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const bool m = (c != 0 && w0) || (c != 1 && w1) || (c != 2 && w2);
    u[c] = m ? T(0) : eo[c];
  }
  T hb[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int a = kAx[c][s], h = kOt[c][s];
      const T sg = s == 0 ? T(1) : T(-1);
      const bool first = c == other0(a);
      // own stencil: d = (H_h(cell) - H_h(cell - e_a)) / dx
      const T w = sg * dt * ei * u[c];
      psib_update(own[a], first, p.psi_out, w);
      hb[h] += dbar(own[a], first, w) * idx;
      // the stencil of the E cell above along a reads H_h(cell) with a minus sign;
      // that cell shares this cell's planes across the other two axes, so the
      // walls through it are those of the other axes (no term beyond a face)
      bool m = false;
#pragma unroll
      for (int b = 0; b < 3; ++b) m = m || (b != a && b != c && wl[b]);
      const T wn = (m || !nb.ok[a]) ? T(0) : sg * dt * epn[a] * en[a][c];
      hb[h] -= dbar(nbr[a], first, wn) * idx;
    }
  if (!OOP && (w0 || w1 || w2)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) p.E[c][id] = u[c];
  }
  const AdjPtrs<T>& d = OOP ? o : p;
#pragma unroll
  for (int c = 0; c < 3; ++c) store_field<NT>(&d.H[c][id], hv[c] + hb[c]);
}

// Transposed H update.  Hb holds the adjoint of H^{n+1/2} (unchanged: identity
// part); Eb gains the curl part.  Out of place, Hb is read from o (the E pass
// wrote it there) and Eb from p, masked on the walls.
template <typename T, bool OOP, bool NT>
__device__ __forceinline__ void adj_h_cell(const AdjPtrs<T>& p, const AdjPtrs<T>& o,
                                           const Geom& g, int i, int j, int k) {
  const size_t id = (size_t)i + (size_t)g.n[0] * ((size_t)j + (size_t)g.n[1] * (size_t)k);
  const T dt = (T)g.dt, idx = (T)g.inv_dx;
  const Nbrs nb = neighbours(g, i, j, k, id, -1);
  const AdjPtrs<T>& hs = OOP ? o : p;
  T hv[3], hn[3][3], ev[3];
#pragma unroll
  for (int h = 0; h < 3; ++h) hv[h] = hs.H[h][id];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int h = 0; h < 3; ++h) hn[a][h] = h != a ? hs.H[h][nb.id[a]] : T(0);
#pragma unroll
  for (int c = 0; c < 3; ++c) ev[c] = p.E[c][id];
  LayerTerm<T> own[3], nbr[3];
  layers_load(g, p, 1, i, j, k, nb, own, nbr);
  if (OOP) {
    const bool w0 = g.wall[0] && i == 0, w1 = g.wall[1] && j == 0, w2 = g.wall[2] && k == 0;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if ((c != 0 && w0) || (c != 1 && w1) || (c != 2 && w2)) ev[c] = T(0);
  }
  T eb[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int h = 0; h < 3; ++h)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int a = kAx[h][s], e = kOt[h][s];
      const T sg = s == 0 ? T(1) : T(-1);
      const bool first = h == other0(a);
      // own stencil: d = (E_e(cell + e_a) - E_e(cell)) / dx, H -= dt sg s(d)
      const T w = -sg * dt * hv[h];
      psib_update(own[a], first, p.psi_out, w);
      eb[e] -= dbar(own[a], first, w) * idx;
      // the stencil of the H cell below along a reads E_e(cell) with a plus sign
      const T wn = nb.ok[a] ? -sg * dt * hn[a][h] : T(0);
      eb[e] += dbar(nbr[a], first, wn) * idx;
    }
  const AdjPtrs<T>& d = OOP ? o : p;
#pragma unroll
  for (int c = 0; c < 3; ++c) store_field<NT>(&d.E[c][id], ev[c] + eb[c]);
}

// The E pass over the cells outside the fused box (out of place: writes o.H), thread t.
template <typename T>
struct AdjShell {
  AdjPtrs<T> p, o;
  ShellMap m;
  int blocks;  // of 256 threads; 0: none
};
template <typename T, bool E_PASS, bool NT>
__device__ __forceinline__ void adj_shell_body(const AdjPtrs<T>& p, const AdjPtrs<T>& o,
                                               const Geom& g, const ShellMap& m, unsigned t) {
  if ((long long)t >= m.total) return;
  int i, j, k;
  shell_cell(g, m, t, i, j, k);
  if (E_PASS) adj_e_cell<T, true, NT>(p, o, g, i, j, k);
  else adj_h_cell<T, true, NT>(p, o, g, i, j, k);
}

}  // namespace mlk
