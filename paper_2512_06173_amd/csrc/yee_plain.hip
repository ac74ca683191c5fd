// Plain (unfused) Yee sweeps: one pass for H, one for E, one thread per cell,
// over a box of cells.
//
// H^{n+1/2} = H^{n-1/2} - dt curl E^n,   E^{n+1} = E^n + (dt/eps_r) curl H^{n+1/2}
// (eq. Maxwell with D = eps_r E, B = H), convolutional PML stretching of each
// spatial derivative inside the absorbing layers, metallic (tangential E = 0)
// or periodic closure.  Source and molecular currents are added by their own
// passes.
//
// The passes read one field buffer (`in`) and write another (`out`); with
// in == out they update in place, which is how the plain sweep runs on the whole
// grid.  The fused sweep uses them, out of place, on the CPML shell: the cells
// outside its interior box, enumerated compactly by one launch per pass.
#include "yee_cells.h"

namespace mlk {

template <typename T, bool H, bool NT>
__global__ __launch_bounds__(256) void k_update_box(FieldPtrs<T> in, FieldPtrs<T> out, Geom g,
                                                    Box box) {
  const int i = box.lo[0] + blockIdx.x * blockDim.x + threadIdx.x;
  const int j = box.lo[1] + blockIdx.y * blockDim.y + threadIdx.y;
  const int k = box.lo[2] + blockIdx.z;
  if (i >= box.hi[0] || j >= box.hi[1]) return;
  if (H) update_h_cell<NT>(in, out, g, i, j, k);
  else update_e_cell<NT>(in, out, g, i, j, k);
}

template <typename T, bool H, bool NT>
__global__ __launch_bounds__(256) void k_update_shell(FieldPtrs<T> in, FieldPtrs<T> out, Geom g,
                                                      ShellMap m) {
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if ((long long)t >= m.total) return;
  int i, j, k;
  shell_cell(g, m, t, i, j, k);
  if (H) update_h_cell<NT>(in, out, g, i, j, k);
  else update_e_cell<NT>(in, out, g, i, j, k);
}

template <typename T, bool H, bool NT>
__global__ __launch_bounds__(256) void k_update_shell_batch(const ShellJob<T>* jobs,
                                                            const int* start, int njobs) {
  const int jb = find_job(start, njobs, blockIdx.x);
  const ShellJob<T> J = load_job(jobs, jb);
  const unsigned t = (blockIdx.x - start[jb]) * blockDim.x + threadIdx.x;
  if ((long long)t >= J.m.total) return;
  int i, j, k;
  shell_cell(J.g, J.m, t, i, j, k);
  if (H) update_h_cell<NT>(J.in, J.out, J.g, i, j, k);
  else update_e_cell<NT>(J.in, J.out, J.g, i, j, k);
}

template <typename T>
__global__ void k_sources(FieldPtrs<T> f, Geom g, SourceSet src, StepNo n) {
  const int q = blockIdx.y;
  if (q >= src.count) return;
  source_body(f, g, src, q, n, blockIdx.x * blockDim.x + threadIdx.x);
}

template <typename T>
__global__ __launch_bounds__(256) void k_sources_batch(const SourceJob<T>* jobs, const int* start,
                                                       int njobs) {
  const int jb = find_job(start, njobs, blockIdx.x);
  const SourceJob<T>& J = jobs[jb];  // (a copy would put its source array in scratch)
  const int lb = blockIdx.x - start[jb];
  if (lb >= J.nblocks) return;
  const int q = lb / J.bx;
  source_body(J.f, J.g, J.src, q, StepNo{J.step, 0}, (lb - q * J.bx) * blockDim.x + threadIdx.x);
}

template <typename T>
static hipError_t launch_plain(const FieldPtrs<T>& in, const FieldPtrs<T>& out, const Geom& g,
                               const Box* boxes, int nbox, bool h_pass, bool e_pass,
                               hipStream_t st) {
  dim3 block(64, 4, 1);
  for (int pass = 0; pass < 2; ++pass) {
    if ((pass == 0 && !h_pass) || (pass == 1 && !e_pass)) continue;
    for (int q = 0; q < nbox; ++q) {
      const Box& b = boxes[q];
      const int ex = b.hi[0] - b.lo[0], ey = b.hi[1] - b.lo[1], ez = b.hi[2] - b.lo[2];
      if (ex <= 0 || ey <= 0 || ez <= 0) continue;
      dim3 grid((ex + 63) / 64, (ey + 3) / 4, ez);
      auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, in, out, g, b); };
      if (pass == 0) g.stream ? go(k_update_box<T, true, true>) : go(k_update_box<T, true, false>);
      else g.stream ? go(k_update_box<T, false, true>) : go(k_update_box<T, false, false>);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

ShellMap shell_map(const Geom& g, const Box& inner) {
  ShellMap m{};
  m.in = inner;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int wy = inner.hi[1] - inner.lo[1], wz = inner.hi[2] - inner.lo[2];
  m.nzlo = inner.lo[2];
  m.nslab = (long long)(nz - wz) * nx * ny;
  m.ylo_rows = inner.lo[1];
  m.full_cells = (ny - wy) * nx;
  m.strip = inner.lo[0] + (nx - inner.hi[0]);
  m.per_plane = m.full_cells + wy * m.strip;
  m.total = m.nslab + (long long)wz * m.per_plane;
  m.inv_plane = 1.0 / ((double)nx * ny);
  m.inv_per_plane = m.per_plane > 0 ? 1.0 / m.per_plane : 0.0;
  m.inv_nx = 1.0 / nx;
  m.inv_strip = m.strip > 0 ? 1.0 / m.strip : 0.0;
  return m;
}

int source_blocks_of(const Geom& g, const SourceSet& src) { return source_blocks(g, src); }

template <typename T>
static hipError_t launch_shell(const FieldPtrs<T>& in, const FieldPtrs<T>& out, const Geom& g,
                               const Box& inner, bool h_pass, hipStream_t st) {
  const ShellMap m = shell_map(g, inner);
  if (m.total == 0) return hipSuccess;
  if (m.total >= 0x7fffff00LL) return hipErrorInvalidValue;  // 32-bit cell index
  const long long blocks = (m.total + 255) / 256;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, in, out, g, m);
  };
  if (h_pass) g.stream ? go(k_update_shell<T, true, true>) : go(k_update_shell<T, true, false>);
  else g.stream ? go(k_update_shell<T, false, true>) : go(k_update_shell<T, false, false>);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_sources(const FieldPtrs<T>& f, const Geom& g, const SourceSet& src,
                                 const StepNo& n, hipStream_t st) {
  if (src.count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sources<T>, dim3(source_blocks(g, src), src.count), dim3(256), 0, st, f, g,
                     src, n);
  return hipGetLastError();
}

hipError_t sweep_plain_f64(const FieldPtrs<double>& in, const FieldPtrs<double>& out,
                           const Geom& g, const Box* boxes, int nbox, bool h_pass, bool e_pass,
                           hipStream_t st) {
  return launch_plain<double>(in, out, g, boxes, nbox, h_pass, e_pass, st);
}
hipError_t sweep_plain_f32(const FieldPtrs<float>& in, const FieldPtrs<float>& out, const Geom& g,
                           const Box* boxes, int nbox, bool h_pass, bool e_pass, hipStream_t st) {
  return launch_plain<float>(in, out, g, boxes, nbox, h_pass, e_pass, st);
}
hipError_t sweep_shell_f64(const FieldPtrs<double>& in, const FieldPtrs<double>& out,
                           const Geom& g, const Box& inner, bool h_pass, hipStream_t st) {
  return launch_shell<double>(in, out, g, inner, h_pass, st);
}
hipError_t sweep_shell_f32(const FieldPtrs<float>& in, const FieldPtrs<float>& out, const Geom& g,
                           const Box& inner, bool h_pass, hipStream_t st) {
  return launch_shell<float>(in, out, g, inner, h_pass, st);
}
template <typename T>
static hipError_t launch_shell_batch(const ShellJob<T>* jobs, const int* start, int njobs,
                                     int nblocks, bool h_pass, bool stream, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(256), 0, st, jobs, start, njobs);
  };
  if (h_pass) stream ? go(k_update_shell_batch<T, true, true>) : go(k_update_shell_batch<T, true, false>);
  else stream ? go(k_update_shell_batch<T, false, true>) : go(k_update_shell_batch<T, false, false>);
  return hipGetLastError();
}
template <typename T>
static hipError_t launch_sources_batch(const SourceJob<T>* jobs, const int* start, int njobs,
                                       int nblocks, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sources_batch<T>, dim3(nblocks), dim3(256), 0, st, jobs, start, njobs);
  return hipGetLastError();
}
hipError_t shell_batch_f64(const ShellJob<double>* jobs, const int* start, int njobs,
                           int nblocks, bool h_pass, bool stream, hipStream_t st) {
  return launch_shell_batch<double>(jobs, start, njobs, nblocks, h_pass, stream, st);
}
hipError_t shell_batch_f32(const ShellJob<float>* jobs, const int* start, int njobs,
                           int nblocks, bool h_pass, bool stream, hipStream_t st) {
  return launch_shell_batch<float>(jobs, start, njobs, nblocks, h_pass, stream, st);
}
hipError_t sources_batch_f64(const SourceJob<double>* jobs, const int* start, int njobs,
                             int nblocks, hipStream_t st) {
  return launch_sources_batch<double>(jobs, start, njobs, nblocks, st);
}
hipError_t sources_batch_f32(const SourceJob<float>* jobs, const int* start, int njobs,
                             int nblocks, hipStream_t st) {
  return launch_sources_batch<float>(jobs, start, njobs, nblocks, st);
}
hipError_t sources_f64(const FieldPtrs<double>& f, const Geom& g, const SourceSet& src,
                       const StepNo& n, hipStream_t st) {
  return launch_sources<double>(f, g, src, n, st);
}
hipError_t sources_f32(const FieldPtrs<float>& f, const Geom& g, const SourceSet& src,
                       const StepNo& n, hipStream_t st) {
  return launch_sources<float>(f, g, src, n, st);
}

}  // namespace mlk
