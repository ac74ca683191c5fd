// Single-mode cavity in place of the grid (Sec. II.A.2: the normal-mode field
// Hamiltonian with the dipole self-energy, its equations of motion and the
// coupling eps = w / sqrt(V) in the single-mode limit, eps0 = 1).
//
// One photonic mode of frequency w with an x and a y polarisation, mode
// function e_l / sqrt(V).  Every emitter feels the same regularised field
//   E~ = -sum_l (eps q_l + d_l / V) e_l,     d_l = sum_m <mu_l^(m)>,
// and the mode obeys q_l'' = -w^2 q_l - eps d_l.  The discretisation follows
// the grid scheme: q at integer steps, p = q' half a step before, emitters at
// half steps.  The total dipole at t_n is the sum of the expectation values of
// the latest states (t_{n-1/2}) carried half a step forward by their own rate,
//   d^n = sum_m [ <mu_m>(rho^{n-1/2}) + (dt/2) mu_dot_m(rho^{n-1/2}) ],
// (eq. dklambda_def at the integer time, second order); mu_dot depends on the
// state alone, so the sum is a function of the states.
//
// A step is one launch per emitter kind.  Its blocks first form the mode at t_n for
// themselves (the same arithmetic in every block): the sum of the partial dipoles that
// the previous step's blocks left, in a fixed order, and the leapfrog of (p, q).  Then
// each thread forms E~, steps its emitter in registers, and the block leaves its
// partial of <mu> + (dt/2) mu_dot of the new states for the next step (two sets in
// turn).  One small launch closes a call of several steps.  A step moves 80 bytes per
// emitter, 2 us for 100,000 at HBM speed; what bounds it is the launch and the chain
// load - sum - sine - sum.  100,000 two-level emitters: 8.8 us a step with the mode
// updated by a launch of its own and the state passed through memory inside the step.
// Beyond kFoldPartials partials (ensembles of several 10,000 multilevel emitters) a
// block of its own adds them up once per step, instead of every block.
// The mode state is six doubles in device memory: q_x, q_y, p_x, p_y, d_x, d_y.
#include "launch.h"
#include "ml_math.h"

namespace mlk {

namespace {

constexpr int kCavThreads = 256;

// Sum of two doubles over the block, in a fixed tree order; the result is
// valid in thread 0.
__device__ __forceinline__ void block_sum2(double& x, double& y) {
  __shared__ double rx[kCavThreads], ry[kCavThreads];
  const int t = threadIdx.x;
  rx[t] = x;
  ry[t] = y;
  __syncthreads();
  for (int w = kCavThreads / 2; w > 0; w >>= 1) {
    if (t < w) {
      rx[t] += rx[t + w];
      ry[t] += ry[t + w];
    }
    __syncthreads();
  }
  x = rx[0];
  y = ry[0];
}

// <mu_x,y> + (dt/2) mu_dot_x,y of every emitter from its state, summed per
// block (two-level slots first, then multilevel slots, each block a fixed
// range).  Two-level: <mu> = 2 Re rho01 d, mu_dot = -2 w0 Im rho01 d.
// Multilevel (mu = d M, rho = R + i I in the zero-padded frame):
// <mu> = d sum_ab R_ab M_ab, mu_dot = d (-2 sum_{a<b} M_ab [I_ab (E_b - E_a) + gphi R_ab]).
__global__ __launch_bounds__(kCavThreads) void k_cavity_partial(TlsPtrs tls, MlDev ml, double dt,
                                                                double* __restrict__ partial) {
  constexpr int F = kMaxLevels;
  const int total = tls.count + ml.count;
  double sx = 0.0, sy = 0.0;
  for (int q = blockIdx.x * kCavThreads + threadIdx.x; q < total; q += gridDim.x * kCavThreads) {
    double mu, rate, dx, dy;
    if (q < tls.count) {
      const double w0 = tls.omega0[q];
      mu = 2.0 * tls.rho[3 * (size_t)q + 1];
      rate = -2.0 * w0 * tls.rho[3 * (size_t)q + 2];
      dx = tls.dip[3 * (size_t)q + 0];
      dy = tls.dip[3 * (size_t)q + 1];
    } else {
      const size_t m = (size_t)(q - tls.count), n = (size_t)ml.count;
      const double g = ml.gphi[m];
      mu = 0.0;
      rate = 0.0;
      for (int a = 0; a < F; ++a) {
        const double ea = ml.en[a * n + m];
        mu += ml.rho[(size_t)(2 * (a * F + a)) * n + m] * ml.M[(size_t)(a * F + a) * n + m];
        for (int b = a + 1; b < F; ++b) {
          const double Mab = ml.M[(size_t)(a * F + b) * n + m];
          const double R = ml.rho[(size_t)(2 * (a * F + b)) * n + m];
          const double I = ml.rho[(size_t)(2 * (a * F + b) + 1) * n + m];
          mu += 2.0 * R * Mab;
          rate += -2.0 * Mab * (I * (ml.en[b * n + m] - ea) + g * R);
        }
      }
      dx = ml.dip[m];
      dy = ml.dip[n + m];
    }
    const double v = mu + 0.5 * dt * rate;
    sx += v * dx;
    sy += v * dy;
  }
  block_sum2(sx, sy);
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x + 0] = sx;
    partial[2 * blockIdx.x + 1] = sy;
  }
}

// Most two-level blocks of a step (each walks the emitters with the grid's stride),
// and the most partials that every block of a step adds up for itself.
constexpr int kTlsBlocks = 1024, kFoldPartials = 1024;

// Sum of the nb partials over one wavefront, in an order that depends on nb alone.
__device__ __forceinline__ void sum_partials(const double* partial, int nb, double& x, double& y) {
  const int lane = threadIdx.x & 63;
  x = 0.0;
  y = 0.0;
  for (int q = lane; q < nb; q += 64) {
    const double2 v = reinterpret_cast<const double2*>(partial)[q];
    x += v.x;
    y += v.y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    x += __shfl_xor(x, off, 64);
    y += __shfl_xor(y, off, 64);
  }
}

// Leapfrog of (p, q) with the old d, then the new d.
__device__ __forceinline__ void mode_advance(const double* old, double dt, double w, double eps,
                                             double dx, double dy, double* st) {
  const double w2 = w * w, d[2] = {dx, dy};
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    const double q = old[l];
    const double p = __builtin_fma(-dt, __builtin_fma(w2, q, eps * old[4 + l]), old[2 + l]);
    st[2 + l] = p;
    st[l] = __builtin_fma(dt, p, q);
    st[4 + l] = d[l];
  }
}

// What the launches of one step share: the mode state of the step before with its
// npend partials (0: `in` is the state of this step), where this step's mode and
// partials go, the step number, and whether E~ and mu_dot are kept (the last step).
struct CavityStep {
  const double* in;
  const double* pend;
  int npend;
  double* out;
  double* partial;
  double dt, w, V, eps;
  StepNo n;
  int last;
};

// E~ of the step, the same for every emitter; the first block of the first launch
// (keep) stores the mode state.
__device__ __forceinline__ void step_field(const CavityStep& c, bool keep, double et[3]) {
  __shared__ double sm[6];
  if (threadIdx.x < 64) {
    double st[6];
    if (c.npend > 0) {
      double dx, dy;
      sum_partials(c.pend, c.npend, dx, dy);
      mode_advance(c.in, c.dt, c.w, c.eps, dx, dy, st);
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) st[k] = c.in[k];
    }
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        sm[k] = st[k];
        if (keep && blockIdx.x == 0) c.out[k] = st[k];
      }
    }
  }
  __syncthreads();
  et[0] = -(c.eps * sm[0] + sm[4] / c.V);
  et[1] = -(c.eps * sm[1] + sm[5] / c.V);
  et[2] = 0.0;
}

// Two-level emitters: the emitter's share of the mode's total dipole at the next
// integer time is <mu> + (dt/2) mu_dot, <mu> = 2 Re rho01 d.
template <int NT>
__global__ __launch_bounds__(NT) void k_cavity_tls(TlsPtrs tls, CavityStep c, double* Et,
                                                   double* mudot, const int64_t* pop_off,
                                                   Series ser) {
  __shared__ double rx[NT / 64], ry[NT / 64];
  const int t = threadIdx.x, stride = gridDim.x * NT;
  int m = blockIdx.x * NT + t;
  // the first emitter's loads are in flight while the mode is formed
  auto load = [&](int k, int& e, double& w0, double d[3], double st[3]) {
    const int q = min(k, tls.count - 1);
    e = tls.gid[q];
    w0 = tls.omega0[q];
    for (int a = 0; a < 3; ++a) {
      d[a] = tls.dip[3 * (size_t)q + a];
      st[a] = tls.rho[3 * (size_t)q + a];
    }
  };
  int e;
  double w0, d[3], st[3], et[3];
  load(m, e, w0, d, st);
  step_field(c, true, et);
  double sx = 0.0, sy = 0.0;
  bool finite = true;
  while (m < tls.count) {
    double md[3];
    tls_advance(w0, d, et, c.dt, st, md);
    finite = finite && isfinite(st[0] + st[1] + st[2] + md[0] + md[1] + md[2]);
    for (int a = 0; a < 3; ++a) tls.rho[3 * (size_t)m + a] = st[a];
    if (c.last)
      for (int a = 0; a < 3; ++a) {
        Et[3 * (size_t)e + a] = et[a];
        mudot[3 * (size_t)e + a] = md[a];
      }
    if (double* pop = pop_record(ser, c.n)) pop[pop_off[e]] = st[0];
    const double mu = 2.0 * st[1];
    sx += mu * d[0] + 0.5 * c.dt * md[0];
    sy += mu * d[1] + 0.5 * c.dt * md[1];
    m += stride;
    if (m < tls.count) load(m, e, w0, d, st);
  }
  if (!finite) flag_nonfinite(ser, c.n.get());
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sx += __shfl_xor(sx, off, 64);
    sy += __shfl_xor(sy, off, 64);
  }
  if ((t & 63) == 0) {
    rx[t >> 6] = sx;
    ry[t >> 6] = sy;
  }
  __syncthreads();
  if (t == 0) {
    for (int k = 1; k < NT / 64; ++k) {
      sx += rx[k];
      sy += ry[k];
    }
    c.partial[2 * blockIdx.x + 0] = sx;
    c.partial[2 * blockIdx.x + 1] = sy;
  }
}

template <int N>
__device__ __forceinline__ void cavity_ml_body(const MlDev& ml, int first, int count,
                                               const CavityStep& c, const double et[3], double* Et,
                                               double* mudot, const int64_t* pop_off,
                                               const Series& ser, int t, double& sx, double& sy) {
  if (t >= count) return;
  const int m = first + t, e = ml.gid[m];
  MlState<N> s;
  ml_load<N>(ml, m, c.dt, s);
  bool finite = true;
  const double tr = ml_advance<N>(s, et, c.dt, finite);
  ml_store<N>(ml, m, s);
  if (c.last)
    for (int a = 0; a < 3; ++a) {
      Et[3 * (size_t)e + a] = et[a];
      mudot[3 * (size_t)e + a] = tr * s.dip[a];
    }
  if (double* pop = pop_record(ser, c.n)) {
    pop += pop_off[e];
#pragma unroll
    for (int a = 1; a < N; ++a) pop[a - 1] = s.R[up<N>(a, a)];
  }
  if (!finite) flag_nonfinite(ser, c.n.get());
  double mu = 0.0;  // sum_ab R_ab M_ab
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = a; b < N; ++b)
      mu += (a == b ? 1.0 : 2.0) * s.R[up<N>(a, b)] * s.M[up<N>(a, b)];
  sx = (mu + 0.5 * c.dt * tr) * s.dip[0];
  sy = (mu + 0.5 * c.dt * tr) * s.dip[1];
}

// Multilevel emitters, every level count in one launch; their partials follow the
// two-level ones.
__global__ __launch_bounds__(64) void k_cavity_ml(MlDev ml, MlLevels lv, CavityStep c, int keep,
                                                  int base, double* Et, double* mudot,
                                                  const int64_t* pop_off, Series ser) {
  double et[3], sx = 0.0, sy = 0.0;
  step_field(c, keep != 0, et);
  const int b = blockIdx.x;
#define MLK_LEVEL(N)                                                                       \
  cavity_ml_body<N>(ml, lv.first[N], lv.count[N], c, et, Et, mudot, pop_off, ser,          \
                    (b - lv.start[N]) * 64 + (int)threadIdx.x, sx, sy)
  if (b < lv.start[5]) MLK_LEVEL(6);
  else if (b < lv.start[4]) MLK_LEVEL(5);
  else if (b < lv.start[3]) MLK_LEVEL(4);
  else if (b < lv.start[2]) MLK_LEVEL(3);
  else MLK_LEVEL(2);
#undef MLK_LEVEL
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sx += __shfl_xor(sx, off, 64);
    sy += __shfl_xor(sy, off, 64);
  }
  if (threadIdx.x == 0) {
    c.partial[2 * (base + b) + 0] = sx;
    c.partial[2 * (base + b) + 1] = sy;
  }
}

// One wavefront: the mode a step on (advance) from the partials, or the new d alone;
// the step counter, when given, moves n steps on.
__global__ __launch_bounds__(64) void k_cavity_mode(const double* in, const double* partial,
                                                    int nb, double dt, double w, double eps,
                                                    int advance, double* out, int64_t* step,
                                                    int64_t n) {
  double dx, dy, old[6], st[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) old[k] = st[k] = in[k];
  sum_partials(partial, nb, dx, dy);
  if (advance) mode_advance(old, dt, w, eps, dx, dy, st);
  st[4] = dx;
  st[5] = dy;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) out[k] = st[k];
    if (step) *step += n;
  }
}

int cavity_blocks(int M) {
  const int nb = (M + 4 * kCavThreads - 1) / (4 * kCavThreads);
  return nb < 1 ? 1 : (nb > kCavThreads ? kCavThreads : nb);
}

// Threads per two-level block: 512, so that every block has few partials to add up
// (100,000 emitters: 6.8 us a step with 256, 5.8 with 512, 6.1 with 1024), 256 where
// the blocks walk the emitters anyway and more of them on a CU hide more (1,000,000:
// 19.5 us with 256, 23.5 with 512).
constexpr int kWideBlocks = 524288;  // emitters up to which a block has 512 threads

int tls_blocks(int count) {
  const int nt = count <= kWideBlocks ? 512 : 256, nb = (count + nt - 1) / nt;
  return nb < kTlsBlocks ? nb : kTlsBlocks;
}

}  // namespace

int cavity_partials(int ntls, const int* ml_range) {
  int mlb = 0;
  (void)ml_levels(ml_range, &mlb);
  const int step = tls_blocks(ntls) + mlb;
  return step > kCavThreads ? step : kCavThreads;  // cavity_set_dipole takes up to 256
}

hipError_t cavity_steps(const CavityDev& cav, const TlsPtrs& tls, const MlDev& ml,
                        const int* range, double dt, int64_t nsteps, double* Et,
                        double* mudot, const int64_t* pop_off, const Series& ser, int64_t* step,
                        hipStream_t st) {
  int mlb = 0;
  const MlLevels lv = ml_levels(range, &mlb);
  const int tb = tls_blocks(tls.count), nb = tb + mlb;
  CavityStep c{};
  c.dt = dt;
  c.w = cav.w;
  c.V = cav.V;
  c.eps = cav.eps;
  c.in = cav.st;
  for (int64_t k = 0; k < nsteps; ++k) {
    // the mode of this step goes to one of the two scratch states in turn (an ensemble
    // that folds nothing keeps it where the mode launch put it)
    c.out = cav.scratch + 6 * (k & 1);
    c.partial = cav.partial + (k & 1) * 2 * (size_t)cav.npart;
    c.n = {step, k};
    c.last = k + 1 == nsteps;
    if (tb > 0 && tls.count <= kWideBlocks)
      hipLaunchKernelGGL(k_cavity_tls<512>, dim3(tb), dim3(512), 0, st, tls, c, Et, mudot, pop_off,
                         ser);
    else if (tb > 0)
      hipLaunchKernelGGL(k_cavity_tls<256>, dim3(tb), dim3(256), 0, st, tls, c, Et, mudot, pop_off,
                         ser);
    if (mlb > 0)
      hipLaunchKernelGGL(k_cavity_ml, dim3(mlb), dim3(64), 0, st, ml, lv, c, tb == 0 ? 1 : 0, tb,
                         Et, mudot, pop_off, ser);
    if (nb > 0 && nb <= kFoldPartials && !c.last) {
      c.in = c.out;
      c.pend = c.partial;
      c.npend = nb;
    } else {  // (no emitters: the mode alone)
      hipLaunchKernelGGL(k_cavity_mode, dim3(1), dim3(64), 0, st, nb > 0 ? c.out : c.in, c.partial,
                         nb, dt, cav.w, cav.eps, 1, cav.st, c.last ? step : nullptr, nsteps);
      c.in = cav.st;
      c.npend = 0;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t cavity_set_dipole(const CavityDev& c, const TlsPtrs& tls, const MlDev& ml, double dt,
                             hipStream_t st) {
  const int M = tls.count + ml.count, nb = M > 0 ? cavity_blocks(M) : 0;
  if (M > 0)
    hipLaunchKernelGGL(k_cavity_partial, dim3(nb), dim3(kCavThreads), 0, st, tls, ml, dt,
                       c.partial);
  hipLaunchKernelGGL(k_cavity_mode, dim3(1), dim3(64), 0, st, c.st, c.partial, nb, dt, c.w, c.eps,
                     0, c.st, nullptr, 0);
  return hipGetLastError();
}

}  // namespace mlk
