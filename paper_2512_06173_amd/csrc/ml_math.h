// Propagator of a multilevel emitter, shared by the coupled, batched and
// classical-path kernels (the model and the splitting are described in
// multilevel.hip).  Everything stays in registers: N, the level count, is a
// template parameter and every loop is unrolled.
#pragma once

#include "tls_math.h"

namespace mlk {

// packed index of the upper triangle (a <= b) of an N x N symmetric matrix
template <int N>
__host__ __device__ constexpr int up(int a, int b) {
  return a <= b ? a * N - a * (a - 1) / 2 + (b - a) : b * N - b * (b - 1) / 2 + (a - b);
}

// Z = X Y for packed symmetric X and Y that commute (polynomials of one matrix): Z is
// symmetric too.
template <int N>
__device__ __forceinline__ void sym_mul(const double (&X)[N * (N + 1) / 2],
                                        const double (&Y)[N * (N + 1) / 2],
                                        double (&Z)[N * (N + 1) / 2]) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = a; b < N; ++b) {
      double z = 0.0;
#pragma unroll
      for (int c = 0; c < N; ++c) z = __builtin_fma(X[up<N>(a, c)], Y[up<N>(c, b)], z);
      Z[up<N>(a, b)] = z;
    }
}

// C = cos A and S = sin A of a packed symmetric A (overwritten), from matrix products only.
// With B = A^2, cos A = p(B) and sin A = A q(B), p and q of degree 7: the polynomials that
// interpolate cos(sqrt y) and sin(sqrt y) / sqrt y at the eight Chebyshev nodes of
// [0, 1.5625] (errors 5e-17 and 3e-18, 1.0e-16 with rounded coefficients), so good for a norm
// up to 1.25.  Seven products: B, B^2, B^3, B^4, one for the upper half of p and of q
// each, and A q.  A larger A is halved s times first and the angle doubled s times after,
// C' = (C - S)(C + S), S' = 2 S C.
// What bounds the kernel is the instruction stream of one wavefront (an emitter per lane,
// few wavefronts on the chip), so operations count: for six levels about 1,200 here, where
// three or four Jacobi sweeps, the sines of the eigenvalues and two products with the
// eigenvectors took 5,000.
template <int N>
__device__ __forceinline__ void cos_sin(double (&A)[N * (N + 1) / 2],
                                        double (&C)[N * (N + 1) / 2],
                                        double (&S)[N * (N + 1) / 2]) {
  constexpr int NS = N * (N + 1) / 2;
  constexpr double p[8] = {1.0, -0.49999999999999584, 0.04166666666661075,
                           -0.0013888888886025015, 2.4801586581049492e-05,
                           -2.755722073848398e-07, 2.0869293481154883e-09,
                           -1.1175623590078535e-11};
  constexpr double q[8] = {1.0, -0.1666666666666664, 0.008333333333330037,
                           -0.00019841269839581692, 2.7557318799284958e-06,
                           -2.5052050342647083e-08, 1.6054646090937375e-10,
                           -7.473341292114921e-13};
  // the largest sum of a row bounds the norm
  double norm = 0.0;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    double r = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) r += fabs(A[up<N>(a, b)]);
    norm = fmax(norm, r);
  }
  // 0.8 norm < 2^s (an infinite norm counts as none: the result is no number either way)
  const int s = max(0, __builtin_amdgcn_frexp_exp(0.8 * norm));
#pragma unroll
  for (int k = 0; k < NS; ++k) A[k] = __builtin_amdgcn_ldexp(A[k], -s);
  {
    double B[NS], B2[NS], B3[NS], B4[NS], t[NS];
    sym_mul<N>(A, A, B);
    sym_mul<N>(B, B, B2);
    sym_mul<N>(B, B2, B3);
    sym_mul<N>(B2, B2, B4);
    auto poly = [&](const double (&c)[8], double (&out)[NS]) {
#pragma unroll
      for (int a = 0; a < N; ++a)
#pragma unroll
        for (int b = a; b < N; ++b) {
          const int k = up<N>(a, b);
          t[k] = __builtin_fma(c[7], B3[k], __builtin_fma(c[6], B2[k], c[5] * B[k])) +
                 (a == b ? c[4] : 0.0);
        }
      sym_mul<N>(B4, t, out);
#pragma unroll
      for (int a = 0; a < N; ++a)
#pragma unroll
        for (int b = a; b < N; ++b) {
          const int k = up<N>(a, b);
          out[k] = __builtin_fma(c[1], B[k], __builtin_fma(c[2], B2[k],
                                                           __builtin_fma(c[3], B3[k], out[k]))) +
                   (a == b ? c[0] : 0.0);
        }
    };
    poly(p, C);
    double u[NS];
    poly(q, u);
    sym_mul<N>(A, u, S);
  }
  for (int k = 0; k < s; ++k) {
    double d[NS], e[NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      d[n] = C[n] - S[n];
      e[n] = C[n] + S[n];
    }
    double c2[NS], s2[NS];
    sym_mul<N>(d, e, c2);
    sym_mul<N>(S, C, s2);
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      C[n] = c2[n];
      S[n] = 2.0 * s2[n];
    }
  }
}

// Every level count in one launch of 64-thread blocks: block b belongs to the level
// count n (from the highest down) whose blocks start at start[n].
struct MlLevels {
  int first[kMaxLevels + 1], count[kMaxLevels + 1], start[kMaxLevels + 1];
};

inline MlLevels ml_levels(const int* range, int* blocks) {
  MlLevels lv{};
  *blocks = 0;
  for (int n = kMaxLevels; n >= 2; --n) {
    lv.first[n] = range[n];
    lv.count[n] = range[n + 1] - range[n];
    lv.start[n] = *blocks;
    *blocks += (lv.count[n] + 63) / 64;
  }
  return lv;
}

// What a multilevel emitter keeps over its steps: the Hamiltonian and the state
// rho = R + i I (R symmetric, I antisymmetric; upper triangles, the diagonal of I
// stays zero).
template <int N>
struct MlState {
  static constexpr int NS = N * (N + 1) / 2;
  double en[N], M[NS], dip[3], gphi, f;  // f: damping of a coherence over half a step
  double R[NS], I[NS];
};

template <int N>
__device__ __forceinline__ void ml_load(const MlDev& ml, int m, double dt, MlState<N>& s) {
  const size_t st = (size_t)ml.count;
  s.gphi = ml.gphi[m];
#pragma unroll
  for (int c = 0; c < 3; ++c) s.dip[c] = ml.dip[c * st + m];
#pragma unroll
  for (int a = 0; a < N; ++a) {
    s.en[a] = ml.en[a * st + m];
#pragma unroll
    for (int b = a; b < N; ++b) {
      const size_t q = (size_t)(a * kMaxLevels + b);
      s.M[up<N>(a, b)] = ml.M[q * st + m];
      s.R[up<N>(a, b)] = ml.rho[(2 * q) * st + m];
      s.I[up<N>(a, b)] = a == b ? 0.0 : ml.rho[(2 * q + 1) * st + m];
    }
  }
  s.f = exp(-0.5 * s.gphi * dt);
}

template <int N>
__device__ __forceinline__ void ml_store(const MlDev& ml, int m, const MlState<N>& s) {
  const size_t st = (size_t)ml.count;
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = a; b < N; ++b) {
      const size_t q = (size_t)(a * kMaxLevels + b), qt = (size_t)(b * kMaxLevels + a);
      const double re = s.R[up<N>(a, b)], im = s.I[up<N>(a, b)];
      ml.rho[(2 * q) * st + m] = re;
      ml.rho[(2 * q + 1) * st + m] = im;
      if (a != b) {
        ml.rho[(2 * qt) * st + m] = re;
        ml.rho[(2 * qt + 1) * st + m] = -im;
      }
    }
}

// One step under the field et: half dephasing, the unitary step, half dephasing.
// Returns Tr(rho_dot M) of the new state (mu_dot = the trace times the dipole);
// finite is cleared when the new populations or the trace are not.
template <int N>
__device__ __forceinline__ double ml_advance(MlState<N>& s, const double et[3], double dt,
                                             bool& finite) {
  constexpr int NS = MlState<N>::NS;
  const double g = et[0] * s.dip[0] + et[1] * s.dip[1] + et[2] * s.dip[2];
  // U = exp(-i H_eff dt) = C - i S (C, S symmetric, packed upper triangles) up to a phase,
  // which leaves U rho U^+ as it is: energies count from the middle of their range
  double C[NS], S[NS];
  {
    double A[NS], lo = s.en[0] - g * s.M[0], hi = lo;
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int b = a; b < N; ++b) {
        const double h = (a == b ? s.en[a] : 0.0) - g * s.M[up<N>(a, b)];
        A[up<N>(a, b)] = h * dt;
        if (a == b) {
          lo = fmin(lo, h);
          hi = fmax(hi, h);
        }
      }
    const double mid = 0.5 * (lo + hi) * dt;
#pragma unroll
    for (int a = 0; a < N; ++a) A[up<N>(a, a)] -= mid;
    cos_sin<N>(A, C, S);
  }
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = a + 1; b < N; ++b) {
      s.R[up<N>(a, b)] *= s.f;
      s.I[up<N>(a, b)] *= s.f;
    }
  auto Rf = [&](int a, int b) { return s.R[up<N>(a, b)]; };
  auto If = [&](int a, int b) {
    return a < b ? s.I[up<N>(a, b)] : (a > b ? -s.I[up<N>(b, a)] : 0.0);
  };
  // rho' = U rho U^+ row by row: T = U rho (row a), rho'_ab = (T U^+)_ab for b >= a;
  // the second half dephasing and the trace follow
  double Rn[NS], In[NS], tr = 0.0, diag = 0.0;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    double Tr_[N], Ti_[N];
#pragma unroll
    for (int b = 0; b < N; ++b) {
      // (C - iS)(R + iI) = (C R + S I) + i (C I - S R)
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const double cac = C[up<N>(a, c)], sac = S[up<N>(a, c)];
        re = __builtin_fma(sac, If(c, b), __builtin_fma(cac, Rf(c, b), re));
        im = __builtin_fma(-sac, Rf(c, b), __builtin_fma(cac, If(c, b), im));
      }
      Tr_[b] = re;
      Ti_[b] = im;
    }
#pragma unroll
    for (int b = a; b < N; ++b) {
      // T (C + iS) with C, S symmetric: column b of C is row b
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const double ccb = C[up<N>(c, b)], scb = S[up<N>(c, b)];
        re = __builtin_fma(-Ti_[c], scb, __builtin_fma(Tr_[c], ccb, re));
        im = __builtin_fma(Ti_[c], ccb, __builtin_fma(Tr_[c], scb, im));
      }
      if (a == b) {
        diag += re;
        In[up<N>(a, b)] = 0.0;
      } else {
        re *= s.f;
        im *= s.f;
        In[up<N>(a, b)] = im;
        tr += s.M[up<N>(a, b)] * (im * (s.en[b] - s.en[a]) + s.gphi * re);
      }
      Rn[up<N>(a, b)] = re;
    }
  }
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    s.R[q] = Rn[q];
    s.I[q] = In[q];
  }
  tr *= -2.0;
  finite = finite && isfinite(tr + diag);
  return tr;
}

}  // namespace mlk
