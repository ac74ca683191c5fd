// Classical-path stepping (eq. E_analytical): emitters under a given field, with no
// grid and no back-action.  No emitter sees another one, so a launch carries each
// emitter through many steps with its parameters and state in registers: per step
// only the field is read (or evaluated) and, when asked for, the state recorded.
// 50 steps of 20,000 two-level and 3,000 multilevel emitters under a pulse: 0.79 ms
// (the six-level emitters' instruction stream), against 3.5 ms with the field, the
// two-level step and five multilevel steps launched at every step.
//
// Two-level emitters: one thread each, bound by the latency of its sine and cosine
// chain.  Multilevel emitters: one thread each (ml_math.h), every level count in one
// launch, the longest first.  When every wavefront of both kinds gets a SIMD of its own,
// the two-level emitters ride in that launch (its registers leave one wavefront a SIMD,
// which is too few for more): 36 us of the 50 steps above.
#include <algorithm>

#include "launch.h"
#include "ml_math.h"
#include "tls_math.h"

namespace mlk {

namespace {

// The field of emitter e over step q of a launch.  wave: a travelling pulse along +z
// at c = 1, gamma amp f(t - (z - z0)) pol with f(u) = cos(omega (u - t0))
// exp(-(u - t0)^2 / (2 tau^2)) (the pulse of App. B), t = t_start + (q0 + q) dt the
// centre of the step; else row q of Et (M x 3 per step, emitter-id order).
__device__ __forceinline__ void field_of(const PrescribedField& f, double dt, int64_t q, int e,
                                         double et[3]) {
  if (f.wave) {
    const double t = f.t_start + (double)(f.q0 + q) * dt;
    const double u = t - (f.pos[3 * (size_t)e + 2] - f.w.z0) - f.w.t0;
    const double a = f.gamma[e] * f.w.amp * cos(f.w.omega * u) *
                     exp(-u * u / (2.0 * f.w.tau * f.w.tau));
    for (int c = 0; c < 3; ++c) et[c] = a * f.w.pol[c];
  } else {
    const double* r = f.Et + (size_t)q * f.stride + 3 * (size_t)e;
    for (int c = 0; c < 3; ++c) et[c] = r[c];
  }
}

__device__ __forceinline__ void tls_run(const TlsPtrs& tls, double dt, const PrescribedField& f,
                                        int nsteps, double* last, double* mudot, double* out,
                                        const Series& ser, const int64_t* step, int m) {
  if (m >= tls.count) return;
  const int e = tls.gid[m];
  const double w0 = tls.omega0[m];
  const double d[3] = {tls.dip[3 * m], tls.dip[3 * m + 1], tls.dip[3 * m + 2]};
  double st[3] = {tls.rho[3 * m], tls.rho[3 * m + 1], tls.rho[3 * m + 2]};
  double md[3] = {0.0, 0.0, 0.0}, et[3] = {0.0, 0.0, 0.0};
  bool finite = true;
  for (int q = 0; q < nsteps; ++q) {
    field_of(f, dt, q, e, et);
    tls_advance(w0, d, et, dt, st, md);
    finite = finite && isfinite(st[0] + st[1] + st[2] + md[0] + md[1] + md[2]);
    if (out) {
      double* o = out + 3 * ((size_t)q * tls.count + m);
      for (int c = 0; c < 3; ++c) o[c] = st[c];
    }
  }
  if (!finite) flag_nonfinite(ser, *step);
  for (int c = 0; c < 3; ++c) {
    tls.rho[3 * m + c] = st[c];
    mudot[3 * e + c] = md[c];
    last[3 * e + c] = et[c];
  }
}

__global__ __launch_bounds__(64) void k_prescribed_tls(TlsPtrs tls, double dt, PrescribedField f,
                                                       int nsteps, double* last, double* mudot,
                                                       double* out, Series ser,
                                                       const int64_t* step) {
  tls_run(tls, dt, f, nsteps, last, mudot, out, ser, step, blockIdx.x * 64 + threadIdx.x);
}

template <int N>
__device__ __forceinline__ void ml_run(const MlDev& ml, int first, int count, double dt,
                                       const PrescribedField& f, int nsteps, double* last,
                                       double* mudot, const Series& ser, const int64_t* step,
                                       int t) {
  if (t >= count) return;
  const int m = first + t, e = ml.gid[m];
  MlState<N> s;
  ml_load<N>(ml, m, dt, s);
  double tr = 0.0, et[3] = {0.0, 0.0, 0.0};
  bool finite = true;
  for (int q = 0; q < nsteps; ++q) {
    field_of(f, dt, q, e, et);
    tr = ml_advance<N>(s, et, dt, finite);
  }
  ml_store<N>(ml, m, s);
  if (!finite) flag_nonfinite(ser, *step);
  for (int c = 0; c < 3; ++c) {
    mudot[3 * e + c] = tr * s.dip[c];
    last[3 * e + c] = et[c];
  }
}

// The blocks from nml on take the two-level emitters.
__global__ __launch_bounds__(64) void k_prescribed_ml(MlDev ml, MlLevels lv, int nml, TlsPtrs tls,
                                                      double dt, PrescribedField f, int nsteps,
                                                      double* last, double* mudot, double* out,
                                                      Series ser, const int64_t* step) {
  const int b = blockIdx.x;
  if (b >= nml) {
    tls_run(tls, dt, f, nsteps, last, mudot, out, ser, step, (b - nml) * 64 + (int)threadIdx.x);
    return;
  }
#define MLK_LEVEL(N)                                                                       \
  ml_run<N>(ml, lv.first[N], lv.count[N], dt, f, nsteps, last, mudot, ser, step,           \
            (b - lv.start[N]) * 64 + (int)threadIdx.x)
  if (b < lv.start[5]) MLK_LEVEL(6);
  else if (b < lv.start[4]) MLK_LEVEL(5);
  else if (b < lv.start[3]) MLK_LEVEL(4);
  else if (b < lv.start[2]) MLK_LEVEL(3);
  else MLK_LEVEL(2);
#undef MLK_LEVEL
}

}  // namespace

// Steps per launch: enough that the launch itself no longer counts, few enough that a
// launch ends within some ten milliseconds.
constexpr int kPrescribedSteps = 256;
constexpr int kSimds = 1024;

hipError_t prescribed_steps(const TlsPtrs& tls, const MlDev& ml, const int* range, double dt,
                            PrescribedField f, int64_t nsteps, double* last, double* mudot,
                            double* out, const Series& ser, const int64_t* step, hipStream_t st) {
  int total = 0;
  const MlLevels lv = ml_levels(range, &total);
  const int ntls = (tls.count + 63) / 64;
  const int ride = total > 0 && total + ntls <= kSimds ? ntls : 0;
  for (int64_t c0 = 0; c0 < nsteps; c0 += kPrescribedSteps) {
    const int k = (int)std::min<int64_t>(kPrescribedSteps, nsteps - c0);
    if (ntls > ride)
      hipLaunchKernelGGL(k_prescribed_tls, dim3(ntls), dim3(64), 0, st, tls, dt, f, k, last, mudot,
                         out, ser, step);
    if (total > 0)
      hipLaunchKernelGGL(k_prescribed_ml, dim3(total + ride), dim3(64), 0, st, ml, lv, total, tls,
                         dt, f, k, last, mudot, out, ser, step);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    f.q0 += k;
    if (f.Et) f.Et += (size_t)k * f.stride;
    if (out) out += (size_t)k * 3 * tls.count;
  }
  return hipSuccess;
}

}  // namespace mlk
