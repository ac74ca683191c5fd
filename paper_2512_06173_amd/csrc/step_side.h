// The short pieces of a step that run as extra workgroups of a larger launch: the
// two-level steps and the closing of the step before (probes, flux total, step
// counter), next to the batched and stand-alone kernels that share the code.
#pragma once

#include "tls_math.h"
#include "yee_cells.h"

namespace mlk {

// Exact two-level step of emitter slot m at step n.
__device__ __forceinline__ void tls_body(const TlsPtrs& tls, double dt, const double* Et,
                                         double* mudot, const int64_t* pop_off, const Series& ser,
                                         const StepNo& n, int m) {
  if (m >= tls.count) return;
  const int e = tls.gid[m];
  const double et[3] = {Et[3 * e], Et[3 * e + 1], Et[3 * e + 2]};
  const double d[3] = {tls.dip[3 * m], tls.dip[3 * m + 1], tls.dip[3 * m + 2]};
  double st[3] = {tls.rho[3 * m], tls.rho[3 * m + 1], tls.rho[3 * m + 2]};
  double md[3];
  tls_advance(tls.omega0[m], d, et, dt, st, md);
  if (!isfinite(st[0] + st[1] + st[2] + md[0] + md[1] + md[2])) flag_nonfinite(ser, n.get());
  tls.rho[3 * m] = st[0];
  tls.rho[3 * m + 1] = st[1];
  tls.rho[3 * m + 2] = st[2];
  mudot[3 * e] = md[0];
  mudot[3 * e + 1] = md[1];
  mudot[3 * e + 2] = md[2];
  if (double* pop = pop_record(ser, n)) pop[pop_off[e]] = st[0];
}

// One workgroup of nt threads (a multiple of 64 up to 1024) closes step n: probe
// samples, the flux total, then the step counter moves on.  The flux partials are
// summed over 256 virtual lanes whatever nt is, so the total does not depend on the
// launch that closes the step.  The counter moves when given (by the last step of a call).
template <typename T>
__device__ __forceinline__ void finish_body(const FieldPtrs<T>& f, const Geom& g,
                                            const FluxPlane& fp, const Series& ser, int64_t n,
                                            int64_t* step, int nt) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  if (t < ser.nprobe) {
    const int comp = ser.probe_comp[t];
    const T* a = comp < 3 ? f.E[comp] : f.H[comp - 3];
    const double v = (double)a[ser.probe_idx[t]];
    if (n < ser.cap) ser.probe[(size_t)t * ser.cap + n] = v;
    if (!isfinite(v)) flag_nonfinite(ser, n);
  }
  if (fp.on) {
    for (int l = t; l < 256; l += nt) {
      double s = 0.0;
      for (int q = l; q < fp.nblocks; q += 256) s += fp.partial[q];
      red[l] = s;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      for (int l = t; l < w; l += nt) red[l] += red[l + w];
      __syncthreads();
    }
    if (t == 0) {
      const double F = red[0] * g.dx * g.dx;
      if (n < ser.cap) fp.series[n] = F;
      *fp.total += g.dt * F;
      if (!isfinite(F)) flag_nonfinite(ser, n);
    }
  }
  __syncthreads();  // every thread may have read n from the counter
  if (t == 0 && step) *step = n + 1;
}

// Extra workgroups of the fused sweep's launch at step n, behind the sweep's own: they
// fill in where its first workgroups end.  They touch nothing that the sweep writes, and it
// reads nothing of theirs: the two-level step works on E~ and the emitter states, step n - 1
// is closed from the fields that the sweep of step n reads, and the shell's H pass reads
// those too and writes cells outside the box.
struct SideWork {
  int blocks;      // workgroups in all (0: none)
  int tls_blocks;  // of these, the first run the two-level step
  int finish;      // 1: the one after them closes step n - 1
  TlsPtrs tls;
  const double* Et;
  double* mudot;
  const int64_t* pop_off;
  Series ser;
  FluxPlane fp;
  StepNo n;
  ShellMap shell;    // H pass over the cells outside the fused box (total 0: none)
};

template <typename T, int NT, bool STREAM>
__device__ __forceinline__ void side_body(const SideWork& w, const FieldPtrs<T>& f,
                                          const FieldPtrs<T>& out, const Geom& g, int b) {
  if (b < w.tls_blocks)
    tls_body(w.tls, g.dt, w.Et, w.mudot, w.pop_off, w.ser, w.n, b * NT + (int)threadIdx.x);
  else if (b < w.tls_blocks + w.finish)
    finish_body(f, g, w.fp, w.ser, w.n.get() - 1, nullptr, NT);
  else {
    const unsigned t = (unsigned)(b - w.tls_blocks - w.finish) * NT + threadIdx.x;
    if ((long long)t >= w.shell.total) return;
    int i, j, k;
    shell_cell(g, w.shell, t, i, j, k);
    update_h_cell<STREAM>(f, out, g, i, j, k);
  }
}

// Workgroup counts of the side work for nt-thread workgroups.
inline void side_blocks(SideWork& w, int nt) {
  w.tls_blocks = (w.tls.count + nt - 1) / nt;
  w.blocks = w.tls_blocks + w.finish + (int)((w.shell.total + nt - 1) / nt);
}

// What else the scatter's launch takes, in workgroups of 256 threads behind its own: the
// flux partials (flux set), and the soft sources (sblocks workgroups each).  Neither may share
// a cell with a window, nor a source with the flux plane.
struct ScatterMore {
  int flux, sblocks;
  FluxPlane fp;
  SourceSet src;
  StepNo n;
};

// What rides in a batch's fused launch: its tables of two-level steps and of shells (for
// their H pass), with the tables' blocks of 256 threads (0: none).
template <typename T>
struct BatchSide {
  const TlsJob* tls;
  const int* tls_start;
  int tls_jobs, ntls;
  const ShellJob<T>* shell;
  const int* shell_start;
  int shell_jobs, nshell;
};

}  // namespace mlk
