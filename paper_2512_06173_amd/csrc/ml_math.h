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

// Cyclic Jacobi (by rows) on the packed symmetric A: A becomes diagonal, Q holds the
// eigenvectors.  The pairs (p, q) of equal p + q are disjoint and wait for none of each
// other, so a sweep of N (N - 1) / 2 rotations goes in 2 N - 3 rounds, whose angles are
// formed side by side:
//   h = sqrt(d^2 + b^2), cos^2 phi = (1 + |d| / h) / 2, t = sgn(d) b / (2 h cos^2 phi),
//   c = 1 / sqrt(t^2 + 1), s = t c,
// d = A_qq - A_pp, b = 2 A_pq (both scaled by a power of two first, so nothing overflows or
// vanishes; reciprocal square roots instead of divisions as far as t).  c keeps the root and
// the quotient of the textbook form: their rounding adds up to 1e-11 in a population over
// 20,000 steps, and what rounds otherwise (c from a reciprocal square root, the same
// rotations in another order, or no rotations: cos and sin of H dt from matrix products,
// whose trace stays within 1e-12) ends up 1.2e-12 to 1.6e-12 apart in the fields and up to
// 2e-11 in the populations, beyond what results are held to.
// Rotations with A_pq = 0 are the identity.  What bounds the kernel is the instruction
// stream of one wavefront (an emitter per lane, few wavefronts on the chip).
template <int N>
__device__ __forceinline__ void jacobi(double (&A)[N * (N + 1) / 2], double (&Q)[N][N]) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) Q[a][b] = a == b ? 1.0 : 0.0;
  for (int sweep = 0; sweep < 32; ++sweep) {
    double off = 0.0, diag = 0.0;
#pragma unroll
    for (int a = 0; a < N; ++a) {
      diag += A[up<N>(a, a)] * A[up<N>(a, a)];
#pragma unroll
      for (int b = a + 1; b < N; ++b) off += A[up<N>(a, b)] * A[up<N>(a, b)];
    }
    if (!(off > 1e-34 * (diag + 2.0 * off))) break;
#pragma unroll
    for (int round = 1; round <= 2 * N - 3; ++round) {
      double cs[N - 1], sn[N - 1], tn[N - 1];
#pragma unroll
      for (int i = 0; i < N - 1; ++i) {
        const int p = i, q = round - i;
        if (q <= p || q >= N) continue;
        const double apq = A[up<N>(p, q)];
        const double d0 = A[up<N>(q, q)] - A[up<N>(p, p)], b0 = 2.0 * apq;
        const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(d0), fabs(b0)));
        const double d = __builtin_amdgcn_ldexp(d0, ex), b = __builtin_amdgcn_ldexp(b0, ex);
        const double rh = rsqrt_refined(__builtin_fma(d, d, b * b));
        const double rc = rsqrt_refined(__builtin_fma(0.5 * fabs(d), rh, 0.5));
        const double t = copysign(0.5, d) * b * rh * rc * rc;
        const double c = 1.0 / sqrt(t * t + 1.0);
        const bool on = apq != 0.0;
        cs[i] = on ? c : 1.0;
        sn[i] = on ? t * c : 0.0;
        tn[i] = on ? t : 0.0;
      }
#pragma unroll
      for (int i = 0; i < N - 1; ++i) {
        const int p = i, q = round - i;
        if (q <= p || q >= N) continue;
        const double c = cs[i], s = sn[i], apq = A[up<N>(p, q)];
        A[up<N>(p, p)] -= tn[i] * apq;
        A[up<N>(q, q)] += tn[i] * apq;
        A[up<N>(p, q)] = 0.0;
#pragma unroll
        for (int r = 0; r < N; ++r) {
          if (r == p || r == q) continue;
          const double arp = A[up<N>(r, p)], arq = A[up<N>(r, q)];
          A[up<N>(r, p)] = c * arp - s * arq;
          A[up<N>(r, q)] = s * arp + c * arq;
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
          const double qrp = Q[r][p], qrq = Q[r][q];
          Q[r][p] = c * qrp - s * qrq;
          Q[r][q] = s * qrp + c * qrq;
        }
      }
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
  // U = exp(-i H_eff dt) = C - i S (C, S symmetric, packed upper triangles)
  double C[NS], S[NS];
  {
    double A[NS], Q[N][N];
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int b = a; b < N; ++b)
        A[up<N>(a, b)] = (a == b ? s.en[a] : 0.0) - g * s.M[up<N>(a, b)];
    jacobi<N>(A, Q);
    double cl[N], sl[N];
#pragma unroll
    for (int q = 0; q < N; ++q) sincos(A[up<N>(q, q)] * dt, &sl[q], &cl[q]);
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int b = a; b < N; ++b) {
        double c = 0.0, v = 0.0;
#pragma unroll
        for (int q = 0; q < N; ++q) {
          const double qq = Q[a][q] * Q[b][q];
          c += qq * cl[q];
          v += qq * sl[q];
        }
        C[up<N>(a, b)] = c;
        S[up<N>(a, b)] = v;
      }
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
