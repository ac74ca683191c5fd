// Multilevel emitters: the open model of Sec. II.B.1 with pure dephasing.
//
// d rho/dt = -i [H_eff, rho] + sum_k (L_k rho L_k^+ - {L_k^+ L_k, rho}/2),
// H_eff = H0 - E~ . mu, H0 = diag(E_0..E_{n-1}), mu^c = d^c M (M real
// symmetric), L_k = sqrt(gphi) |k><k|   (eq. von-Neumann-tls with the
// Lindblad term).
//
// One step over dt (Strang splitting, second order):
//   dephase(dt/2): rho_ab *= exp(-gphi dt/2) for a != b   (exact for this dissipator)
//   unitary:       rho <- U rho U^+, U = exp(-i H_eff dt) = C - i S,
//                  C = Q cos(L dt) Q^T, S = Q sin(L dt) Q^T from H_eff = Q L Q^T
//   dephase(dt/2)
// then mu_dot^c = Tr(rho_dot mu^c) (eq. dipole_derivative) at the new state.  For
// this model the trace has a closed form (with rho = R + i I):
//   Tr(rho_dot M) = -2 sum_{a<b} M_ab [ I_ab (E_b - E_a) + gphi R_ab ]
// (the field term drops out because [M, M] = 0; the dissipator only damps
// the coherences).  For n = 2 it reduces to the two-level -2 w0 Im rho01.
//
// One thread per emitter, the level count n a template parameter so that every
// matrix lives in registers (ml_math.h).  State is stored structure-of-arrays
// (entry-major) so that neighbouring threads read neighbouring words.
//
// Emitters are grouped by n.  What bounds the step is the FP64 instruction stream of
// a lone wavefront per SIMD (10,000 emitters are 159 wavefronts for 1024 SIMDs), so
// the groups of a mixed ensemble run side by side in one launch, the longest first,
// instead of one launch after another: 10,000 emitters of 2 to 6 levels took
// 25.6 + 17.5 + 11.6 + 7.2 + 4.9 us in five launches, 18.8 in one with the rotations of a
// round side by side (ml_math.h).
#include "ml_math.h"

namespace mlk {

// Mixed ensembles of at most this many wavefronts take one launch.  It runs one
// wavefront per SIMD (the registers of six levels); separate launches give the small
// level counts more, which could only tell where a level count fills the chip by
// itself.  Measured, separate against one launch, a step of 64^3 cells with 1,000,
// 10,000, 50,000 and 200,000 emitters of 2 to 6 levels: 66.1, 72.8, 101.6, 191.3 against
// 37.3, 43.5, 71.1, 164.4 us.
constexpr int kMlOneLaunchBlocks = 8192;

template <int N>
__device__ __forceinline__ void ml_body(const MlDev& ml, int first, int count, double dt,
                                        const double* Et, double* mudot, const int64_t* pop_off,
                                        const Series& ser, const StepNo& n, int t) {
  const int m = first + t;
  if (t >= count) return;
  const int e = ml.gid[m];
  MlState<N> s;
  ml_load<N>(ml, m, dt, s);
  const double et[3] = {Et[3 * e], Et[3 * e + 1], Et[3 * e + 2]};
  bool finite = true;
  const double tr = ml_advance<N>(s, et, dt, finite);
  ml_store<N>(ml, m, s);
  if (double* pop = pop_record(ser, n)) {
    pop += pop_off[e];
#pragma unroll
    for (int a = 1; a < N; ++a) pop[a - 1] = s.R[up<N>(a, a)];
  }
  if (!finite) flag_nonfinite(ser, n.get());
#pragma unroll
  for (int c = 0; c < 3; ++c) mudot[3 * e + c] = tr * s.dip[c];
}

template <int N>
__global__ __launch_bounds__(64) void k_ml_step(MlDev ml, int first, int count, double dt,
                                                const double* Et, double* mudot,
                                                const int64_t* pop_off, Series ser, StepNo n) {
  ml_body<N>(ml, first, count, dt, Et, mudot, pop_off, ser, n,
             blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(64) void k_ml_levels(MlDev ml, MlLevels lv, double dt,
                                                  const double* Et, double* mudot,
                                                  const int64_t* pop_off, Series ser,
                                                  StepNo n) {
  const int b = blockIdx.x;
#define MLK_LEVEL(N)                                                                  \
  ml_body<N>(ml, lv.first[N], lv.count[N], dt, Et, mudot, pop_off, ser, n,            \
             (b - lv.start[N]) * 64 + (int)threadIdx.x)
  if (b < lv.start[5]) MLK_LEVEL(6);
  else if (b < lv.start[4]) MLK_LEVEL(5);
  else if (b < lv.start[3]) MLK_LEVEL(4);
  else if (b < lv.start[2]) MLK_LEVEL(3);
  else MLK_LEVEL(2);
#undef MLK_LEVEL
}

template <int N>
__global__ __launch_bounds__(64) void k_ml_batch(const MlJob* jobs, const int* start, int njobs) {
  const int j = find_job(start, njobs, blockIdx.x);
  const MlJob J = load_job(jobs, j);
  const int lb = blockIdx.x - start[j];
  if (lb >= J.nblocks) return;
  ml_body<N>(J.ml, J.first, J.count, J.dt, J.Et, J.mudot, J.pop_off, J.ser, StepNo{J.step, 0},
             lb * blockDim.x + threadIdx.x);
}

// Batched multilevel step; every job of the table has `nl` levels.
hipError_t ml_batch(const MlJob* jobs, const int* start, int njobs, int nblocks, int nl,
                    hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  const dim3 grid(nblocks), block(64);
  switch (nl) {
    case 2: hipLaunchKernelGGL(k_ml_batch<2>, grid, block, 0, st, jobs, start, njobs); break;
    case 3: hipLaunchKernelGGL(k_ml_batch<3>, grid, block, 0, st, jobs, start, njobs); break;
    case 4: hipLaunchKernelGGL(k_ml_batch<4>, grid, block, 0, st, jobs, start, njobs); break;
    case 5: hipLaunchKernelGGL(k_ml_batch<5>, grid, block, 0, st, jobs, start, njobs); break;
    case 6: hipLaunchKernelGGL(k_ml_batch<6>, grid, block, 0, st, jobs, start, njobs); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t ml_step(const MlDev& ml, const int* range, double dt, const double* Et, double* mudot,
                   const int64_t* pop_off, const Series& ser, const StepNo& n, hipStream_t st) {
  int total = 0;
  const MlLevels lv = ml_levels(range, &total);
  if (total == 0) return hipSuccess;
  int kinds = 0;
  for (int nl = 2; nl <= kMaxLevels; ++nl) kinds += lv.count[nl] > 0;
  if (kinds > 1 && total <= kMlOneLaunchBlocks) {
    hipLaunchKernelGGL(k_ml_levels, dim3(total), dim3(64), 0, st, ml, lv, dt, Et, mudot, pop_off,
                       ser, n);
    return hipGetLastError();
  }
  for (int nl = 2; nl <= kMaxLevels; ++nl) {
    const int first = lv.first[nl], count = lv.count[nl];
    if (count <= 0) continue;
    const dim3 grid((count + 63) / 64), block(64);
    switch (nl) {
      case 2: hipLaunchKernelGGL(k_ml_step<2>, grid, block, 0, st, ml, first, count, dt, Et, mudot, pop_off, ser, n); break;
      case 3: hipLaunchKernelGGL(k_ml_step<3>, grid, block, 0, st, ml, first, count, dt, Et, mudot, pop_off, ser, n); break;
      case 4: hipLaunchKernelGGL(k_ml_step<4>, grid, block, 0, st, ml, first, count, dt, Et, mudot, pop_off, ser, n); break;
      case 5: hipLaunchKernelGGL(k_ml_step<5>, grid, block, 0, st, ml, first, count, dt, Et, mudot, pop_off, ser, n); break;
      case 6: hipLaunchKernelGGL(k_ml_step<6>, grid, block, 0, st, ml, first, count, dt, Et, mudot, pop_off, ser, n); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mlk
