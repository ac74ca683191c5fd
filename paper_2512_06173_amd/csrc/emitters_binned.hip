// Two-level steps and current scatter of the binned emitter phase (the gather is in
// gather.hip).
//
// step (eq. von-Neumann-tls, eq. dipole_derivative): one thread per two-level
// emitter advances its state with the exact propagator and writes mu_dot.
//
// scatter (eqs. J_mol, Polarization_mol):  E_c(p) -= (dt/eps_r(p)) gamma mu_dot^c
// w^c_{m,p} / dx^3.  A wavefront owns a bin of cells and takes every (emitter,
// bin) pair whose window touches the bin, on the matrix cores (see scatter_body);
// each cell is written once by its owner (no atomics, a fixed order of sums).
//
// Window weights are the separable factors wx wy wz set up by k_windows, kept
// per emitter as a union-window record (WinRec); a component uses the
// half-integer variant on its own axis.
#include "launch.h"

namespace mlk {

void bin_shape(bool fp32, int G[3], int S[3]) {
  gather_bin_shape(fp32, G);
  S[0] = kScX; S[1] = kScY; S[2] = kScZ;
}

// A wavefront takes 0.7 us for a chunk of pairs, whatever else the chip does, so a bin of many
// pairs that a wavefront had to itself kept the launch waiting; sharing costs a bin of few pairs
// the exchange.  Limits of 64, 128, 256 and 512 pairs, us: FP32 128^3 with 100,000 emitters
// 45.7, 36.1, 35.9, 36.6; 10,000 in 12 planes of 64 x 64 12.3, 13.4, 18.7, 26.4; 300 within four
// cells 9.8, 10.7, 10.9, 20.3; FP64 86.7, 69.6, 70.3, 71.5; 17.5, 19.4, 30.2, 44.3; 13.1, 13.8,
// 13.8, 33.5.
int scatter_shared() { return 128; }

// Every pair of an emitter fetches its gamma and mu_dot, 8.6 times in all, and in the emitters'
// own order each time from some other line; beyond what an L2 holds these trips weigh more than
// the rest.  Larger ensembles put the amplitudes in the gather's order first, where those of
// a bin's pairs lie together.  In 128^3 cells, us without and with: FP32 100,000 emitters 39.0,
// 40.9; 200,000 75.5, 75.9; 300,000 112.9, 98.8; 1,000,000 504, 351; FP64 200,000 143, 147;
// 300,000 185, 193; 1,000,000 687, 545.
int scatter_amps_min(bool fp32) { return fp32 ? 262144 : 524288; }

__global__ __launch_bounds__(256) void k_scatter_amps(BinPtrs bins, const double* gamma,
                                                      const double* a, double amp0) {
  const unsigned t = blockIdx.x * 256u + threadIdx.x, q = t / 3u;
  if (q >= (unsigned)bins.nem) return;
  const int e = bins.gbin_em[q];
  bins.amp[t] = amp0 * gamma[e] * a[3 * (size_t)e + (t - 3u * q)];
}

hipError_t scatter_amps(const BinPtrs& b, const double* gamma, const double* a, double amp0,
                        hipStream_t st) {
  if (!b.amp || b.nem <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)(((size_t)3 * b.nem + 255) / 256);
  hipLaunchKernelGGL(k_scatter_amps, dim3(blocks), dim3(256), 0, st, b, gamma, a, amp0);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_tls_step(TlsPtrs tls, double dt, const double* Et,
                                                  double* mudot, const int64_t* pop_off,
                                                  Series ser, StepNo n) {
  tls_body(tls, dt, Et, mudot, pop_off, ser, n, blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(256) void k_tls_batch(const TlsJob* jobs, const int* start,
                                                   int njobs) {
  const int j = find_job(start, njobs, blockIdx.x);
  const TlsJob J = load_job(jobs, j);
  const int lb = blockIdx.x - start[j];
  if (lb >= J.nblocks) return;
  tls_body(J.tls, J.dt, J.Et, J.mudot, J.pop_off, J.ser, StepNo{J.step, 0},
           lb * blockDim.x + threadIdx.x);
}

namespace {

template <typename T>
struct ScatterCfg {
  static constexpr int pairs = sizeof(T) == 4 ? 16 : 8;   // of a chunk
  static constexpr int waves = sizeof(T) == 4 ? 5 : 3;  // per SIMD
};
constexpr int kThreads = 64 * kScWaves;

// v_mfma 16 x 16 x 4: D[i][j] += sum_k A[i][k] B[k][j]; lane l gives A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds four rows of column l % 16: rows 4 (l / 16) + r of a FP32
// product, rows l / 16 + 4 r of a FP64 one.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  using Acc = f32x4;
  __device__ static Acc madd(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int k, int r) { return 4 * k + r; }
};
template <>
struct Mfma<double> {
  using Acc = f64x4;
  __device__ static Acc madd(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int k, int r) { return k + 4 * r; }
};

}  // namespace

// scatter; see the file comment.  E_c(p) -= [eps_r^-1(p) if EPS] amp0 gamma a^c w^c_p over
// the windows, with a = mudot (the forward current: amp0 = dt / dx^3, EPS) or any other
// per-emitter amplitude (the adjoint step: amp0 = -1, no EPS).
//
// The weights are products wx wy wz, so the current of a bin is a matrix product over
// its pairs m, per component c:
//   J_c[(y, z), x] = sum_m (wy_m(y) wz_m(z)) (amp_m^c wx_m(x)).
// A wavefront owns a bin of 16 x by 4 y and 4 z (16 rows) and takes its pairs four at a
// time, three 16 x 16 x 4 products of the field's own precision each.  A bin of many pairs (see
// scatter_shared) is shared by the four wavefronts of a workgroup, a quarter of the pairs each,
// whose sums are added in FP64 and in order: 10,000 emitters within four cells 442 -> 117 us
// (FP64 847 -> 220), 10,000 in 12 planes of 64 x 64 26.6 -> 13.6 (43 -> 19).
//
// A pair (emitter, bin) comes with its offset per axis, set up on the host (see
// PairDesc): bin-local cell x reads weight x + o.  The weights are staged in LDS with
// zeros around the eight of y and z, and one behind those of x for every offset beside
// them, so there are no bounds checks.  A window that wraps inside one bin (a periodic axis
// no longer than the bin) is split into several pairs.  What a pair reads beside its run
// of cells is zero: a run begins at weight 0 or at cell 0, and ends with the weights, with
// the bin or with the axis, whose cells are the only ones written.
//
// Otherwise the wavefronts of a workgroup share nothing and never wait for each other; registers allow
// five a SIMD (FP64: three), which hide the trips to memory of each other (ids, then records, then
// E).  With 50,000 to 100,000 emitters no unit is busy more than a third of the time (cube:
// VALU 32%, matrix cores 18%, LDS 27%) and the reads and writes of E run at 1 to 4 TB/s: what
// is left is latency.  Before, a workgroup of eight wavefronts summed a bin of 16 x 16 x 16
// (8 with FP64) cells with LDS atomics, two or three per cell and emitter.  Kernel times,
// us a step, before and now: cube 256^3 with 100,000 emitters 59.6 -> 50, 187 x 149 x 163
// FP64 with 20,000 76 -> 53, 384^3 with 100,000 113 -> 89, 160^3 with 10,000 28 -> 16.7,
// 1,000 in 128^3 10.4 -> 6.1.  Measured and not taken: bins of four wavefronts with
// their pairs staged together (cube 51, 64 x 64 planes 36); E read at the start (54).
//
// Blocks from bins.nscatter on (when more is given) form the flux partials of the plane, in
// the LDS of the weights, and then the soft sources.
// AMPS: amplitudes in the gather's order where the bins have them (see scatter_amps).
template <typename T, bool AMPS, bool EPS = true>
__device__ __forceinline__ void scatter_body(const FieldPtrs<T>& f, const Geom& g,
                                             const BinPtrs& bins, const WindowPtrs<T>& win,
                                             const double* mudot, double amp0, int bid,
                                             const ScatterMore* more = nullptr) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  typedef int piece_t __attribute__((ext_vector_type(4)));
  using M = Mfma<T>;
  constexpr int P = ScatterCfg<T>::pairs;
  // FP32 amplitudes are held 2^-9 of what they are: the largest weight of a window is at least
  // 8^-3, so an amplitude beyond what is left (which counts as the limit: an infinity would
  // spoil the bin) exceeds FP32 in its window
  constexpr double kAmpScale = sizeof(T) == 4 ? 0x1p-9 : 1.0;
  constexpr float kAmpMax = 3.4028234663852886e38f;
  // a pair's weights in LDS: x at 0, y at kY, z at kZ, zeros between and behind
  constexpr int kY = 12, kZ = 24, kStride = 36;
  constexpr int kPer = 16 / (int)sizeof(T2);   // weights per 16-byte piece
  constexpr int R4 = 3 * kMaxWin / kPer;       // pieces of a record
  constexpr int NP = P * R4 / 64;              // pieces per lane and chunk
  static_assert(P * R4 % 64 == 0 && 3 * P <= 64 && P % 4 == 0 && kMaxWin == 8, "chunk");
  // (or, of a bin that the workgroup shares, the wavefronts' sums: 12 a lane)
  constexpr int kWin = P * kStride > 12 * 64 / 2 ? P * kStride : 12 * 64 / 2;
  __shared__ alignas(16) T2 sWin[kScWaves][kWin];
  __shared__ alignas(16) T sAmp[kScWaves][P][4];
  __shared__ int sOff[kScWaves][P];
  __shared__ double sTot[3][kThreads];
  __shared__ float sRem[sizeof(T) == 8 ? kScWaves * 12 * 64 : 1];
  if (more && bid >= bins.nscatter) {  // uniform across the block
    static_assert(sizeof(sWin) >= 256 * sizeof(double) && kThreads == 256, "the flux sums");
    int b = bid - bins.nscatter;
    const int nflux = more->flux ? more->fp.nblocks : 0;
    if (b < nflux) {
      flux_partial_sum(f, g, more->fp, b, nflux, reinterpret_cast<double*>(&sWin[0][0]));
    } else {
      b -= nflux;
      const int q = b / more->sblocks;
      source_body(f, g, more->src, q, more->n, (b - q * more->sblocks) * 256 + threadIdx.x);
    }
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int4 bin = bins.sbin[bid * kScWaves + wave];
  if (bin.y >= bin.z) return;  // fills up the last workgroup
  const bool shared = bin.w != 0;  // uniform across the workgroup
  int q0 = bin.y, q1 = bin.z;
  // A shared bin's pairs go in rounds of an equal part for each wavefront: in FP32 of at
  // most kChain pairs, as the sums of a round are added up in FP64 (sTot: of the row that the
  // thread writes), so that the error of J does not grow with the emitters around a cell
  // (5.4e-8 of the largest, rms, with 128, 1.9e-8 with 4,000; 2.9e-7 without rounds; 10,000
  // emitters within four cells 117 -> 127 us); in FP64 in one round, the rounding errors of
  // whose sums are kept (sRem).
  constexpr int kChain = 256;
  int rounds = 1, quarter = 0;
  if (shared) {
    if (sizeof(T) == 4) rounds = (q1 - q0 + kScWaves * kChain - 1) / (kScWaves * kChain);
    const int step = kScWaves * P * rounds;
    quarter = (q1 - q0 + step - 1) / step * P;
    q0 = min(bin.y + wave * quarter, bin.z);
    q1 = min(q0 + quarter, bin.z);
  }

  // A chunk's weights and amplitudes pass through registers: its loads are issued a
  // chunk ahead, those of the emitters, on which they depend, two chunks ahead.
  int slot[NP], part[NP], rec[NP];
  int2 apd = make_int2(0, 0);
  int aoff = 0;
  piece_t piece[NP];
  double pg = 1.0, pm = 0.0;
  const int apair = lane / 3, acomp = lane % 3;  // lanes below 3 P: a pair's amplitudes
  const bool ordered = AMPS && bins.amp;
  const double* const amps = ordered ? bins.amp : mudot;
  const double scale = (ordered ? 1.0 : amp0) * kAmpScale;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    slot[p] = (lane + p * 64) / R4;
    part[p] = (lane + p * 64) % R4;
  }
  auto load_pairs = [&](int c) {
#pragma unroll
    for (int p = 0; p < NP; ++p) rec[p] = bins.sbin_pair[min(c + slot[p], q1 - 1)].z;
    apd = *reinterpret_cast<const int2*>(&bins.sbin_pair[min(c + min(apair, P - 1), q1 - 1)]);
  };
  auto load_records = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p)
      piece[p] = reinterpret_cast<const piece_t*>(win.rec)[(unsigned)(rec[p] + part[p])];
    aoff = apd.y;
    if (!ordered) pg = win.gamma[apd.x];
    pm = amps[3 * apd.x + acomp];
  };
  auto begin = [&] {
    load_pairs(q0);
    int t = lane;
    asm("" : "+v"(t));  // (formed anew in every round, not kept in registers)
    for (; t < P * kStride * (int)sizeof(T2) / 16; t += 64)
      reinterpret_cast<piece_t*>(&sWin[wave][0])[t] = piece_t{0, 0, 0, 0};
    load_records();
    if (q0 + P < q1) load_pairs(q0 + P);
  };
  const int lx = lane & 15, lk = lane >> 4;  // column (and row of A), pair of a step
  const int yl = kY + (lx & 3), zl = kZ + (lx >> 2);
  typename M::Acc acc[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) acc[c] = {0, 0, 0, 0};
  auto stage = [&](int cn) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int axis = part[p] * kPer / kMaxWin, d = part[p] * kPer % kMaxWin;
      *reinterpret_cast<piece_t*>(&sWin[wave][slot[p] * kStride + kY * axis + d]) = piece[p];
    }
    if (lane < 3 * P) {
      // an amplitude that is no number adds nothing (times the zeros beside its window
      // it would spoil the whole bin), nor does what fills up the last step
      const double v = scale * pg * pm;
      T a = (T)v;
      if constexpr (sizeof(T) == 4) a = __builtin_amdgcn_fmed3f(a, -kAmpMax, kAmpMax);
      sAmp[wave][apair][acomp] = apair < cn && fabs(v) <= 1.7976931348623157e308 ? a : T(0);
      if (acomp == 0) sOff[wave][apair] = aoff;
    }
  };
  // (the LDS serves a wavefront in order; the fences keep the compiler's order)
  auto order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto sums = [&](int cn) {
    order();
#pragma unroll
    for (int s = 0; s < P; s += 4) {
      if (s >= cn) break;
      const int m = s + lk, o = sOff[wave][m];
      const T2* w = &sWin[wave][m * kStride];
      const unsigned ix = (unsigned)(lx + (int)(signed char)o);
      const T2 wx = w[ix < 8u ? ix : 8u];
      const T2 wy = w[yl + (int)(signed char)(o >> 8)];
      const T2 wz = w[zl + (int)(signed char)(o >> 16)];
      const T* am = sAmp[wave][m];
      // a component takes the half-integer weights on its own axis
      acc[0] = M::madd(wy.x * wz.x, am[0] * wx.y, acc[0]);
      acc[1] = M::madd(wy.y * wz.x, am[1] * wx.x, acc[1]);
      acc[2] = M::madd(wy.x * wz.y, am[2] * wx.x, acc[2]);
    }
    order();
  };
  // FP64: the sums of a chunk are added to those of the chunks before with the rounding
  // error of the addition kept (Knuth's two-sum), as exact as a wider accumulator: with
  // 256 emitters around one cell the error of J is 2.2e-16 (rms), 5.6e-16 without; the
  // registers cost a wavefront per SIMD, not time (54 -> 53 us)
  constexpr bool kExact = sizeof(T) == 8;
  typename M::Acc hi[kExact ? 3 : 1], lo[kExact ? 3 : 1];
  auto fold = [&] {
    if constexpr (kExact) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const typename M::Acc t = hi[c] + acc[c], b = t - hi[c];
        lo[c] += (hi[c] - (t - b)) + (acc[c] - b);
        hi[c] = t;
        acc[c] = {0, 0, 0, 0};
      }
    }
  };
  if constexpr (kExact) {
#pragma unroll
    for (int c = 0; c < 3; ++c) hi[c] = lo[c] = {0, 0, 0, 0};
  }
  int c0;
  auto chunks = [&] {  // all, but for the last one's sums
    for (c0 = q0; c0 + P < q1; c0 += P) {
      stage(P);
      load_records();
      if (c0 + 2 * P < q1) load_pairs(c0 + 2 * P);
      sums(P);
      fold();
    }
    if (c0 < q1) stage(q1 - c0);
  };
  // the wavefronts' sums of a round into sTot, in their order
  auto add_round = [&](bool first) {
    if (c0 < q1) sums(q1 - c0);
    if constexpr (kExact) fold();
    __syncthreads();
    T* s = reinterpret_cast<T*>(&sWin[0][0]);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = ((wave * 3 + c) * 4 + r) * 64 + lane;
        T v = acc[c][r];
        if constexpr (kExact) {
          v = hi[c][r] + lo[c][r];
          sRem[o] = (float)((hi[c][r] - v) + lo[c][r]);
        }
        s[o] = v;
      }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double tot = first ? 0.0 : sTot[c][threadIdx.x], err = 0.0;
#pragma unroll
      for (int w = 0; w < kScWaves; ++w) {
        const int o = ((w * 3 + c) * 4 + wave) * 64 + lane;
        const double v = (double)s[o], t = tot + v;
        if constexpr (kExact) {
          const double b = t - tot;
          err += (tot - (t - b)) + (v - b) + (double)sRem[o];
        }
        tot = t;
      }
      sTot[c][threadIdx.x] = tot + err;
    }
  };
  for (int k = 1;; ++k) {
    begin();
    chunks();
    if (k >= rounds) break;
    add_round(k == 1);
    __syncthreads();
    q0 = min(bin.y + (k * kScWaves + wave) * quarter, bin.z);
    q1 = min(q0 + quarter, bin.z);
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = {0, 0, 0, 0};
  }
  // Lane l holds x = l % 16 and four of the rows (y, z), neighbours along y (FP32) or z
  // (FP64), nr of them in the grid.  Their E is read ahead of the last chunk's sums.
  const int bx = bin.x % bins.nbx, by = (bin.x / bins.nbx) % bins.nby,
            bz = bin.x / (bins.nbx * bins.nby);
  const int row = M::row(lk, 0);
  const int x = kScX * bx + lx, y = kScY * by + (row & 3), z = kScZ * bz + (row >> 2);
  const size_t step = sizeof(T) == 4 ? (size_t)g.n[0] : (size_t)g.n[0] * g.n[1];
  const size_t cell = cell_index(g, x, y, z);
  const int nr = x < g.n[0] && y < g.n[1] && z < g.n[2]
                     ? min(4, sizeof(T) == 4 ? g.n[1] - y : g.n[2] - z)
                     : 0;
  T ev[4][3], ei[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    ei[r] = T(1);
#pragma unroll
    for (int c = 0; c < 3; ++c) ev[r][c] = r < nr ? f.E[c][cell + r * step] : T(0);
    if (EPS && f.epsinv && r < nr) ei[r] = f.epsinv[cell + r * step];  // null: eps_r = 1
  }
  if (shared) {  // wavefront r writes row r
    add_round(rounds == 1);
    const bool in = wave < nr;
    const size_t own = cell + wave * step;
    T e[3], ei = T(1);
#pragma unroll
    for (int c = 0; c < 3; ++c) e[c] = in ? f.E[c][own] : T(0);
    if (EPS && f.epsinv && in) ei = f.epsinv[own];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double v = sTot[c][threadIdx.x];
      if (in && v != 0.0) f.E[c][own] = e[c] - ei * (T)(v / kAmpScale);
    }
    return;
  }
  sums(q1 - c0);
  if constexpr (kExact) {
    fold();
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = hi[c] + lo[c];
  }
  // owner write: E -= [eps^-1] J
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (r < nr && acc[c][r] != T(0))
        f.E[c][cell + r * step] = ev[r][c] - ei[r] * (acc[c][r] * T(1 / kAmpScale));
}

template <typename T, bool AMPS>
__global__ __launch_bounds__(kThreads, ScatterCfg<T>::waves) void k_scatter_bins(
    FieldPtrs<T> f, Geom g, BinPtrs bins, WindowPtrs<T> win, const double* mudot) {
  scatter_body<T, AMPS>(f, g, bins, win, mudot, g.dt * g.inv_dx * g.inv_dx * g.inv_dx, blockIdx.x);
}

// The scatter with the flux partials and the soft sources in more workgroups.
template <typename T, bool AMPS>
__global__ __launch_bounds__(kThreads, ScatterCfg<T>::waves) void k_scatter_more(
    FieldPtrs<T> f, Geom g, BinPtrs bins, WindowPtrs<T> win, const double* mudot,
    ScatterMore more) {
  scatter_body<T, AMPS>(f, g, bins, win, mudot, g.dt * g.inv_dx * g.inv_dx * g.inv_dx, blockIdx.x,
                        &more);
}

template <typename T, bool AMPS>
__global__ __launch_bounds__(kThreads, ScatterCfg<T>::waves) void k_scatter_batch(
    const ScatterJob<T>* jobs, const int* start, int njobs, const int2* order) {
  int j, bid;
  if (order) {  // (job, block) of the block, heaviest first across the jobs
    const int2 o = order[blockIdx.x];
    j = o.x;
    bid = o.y;
  } else {
    j = find_job(start, njobs, blockIdx.x);
    bid = blockIdx.x - start[j];
    if (bid >= jobs[j].nblocks) return;
  }
  const ScatterJob<T> J = load_job(jobs, j);
  scatter_body<T, AMPS>(J.f, J.g, J.bins, J.win, J.mudot,
                        J.g.dt * J.g.inv_dx * J.g.inv_dx * J.g.inv_dx, bid);
}

hipError_t tls_step(const TlsPtrs& tls, double dt, const double* Et, double* mudot,
                    const int64_t* pop_off, const Series& ser, const StepNo& n, hipStream_t st) {
  if (tls.count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tls_step, dim3((tls.count + 255) / 256), dim3(256), 0, st, tls, dt, Et,
                     mudot, pop_off, ser, n);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_scatter(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                                 const WindowPtrs<T>& win, const double* mudot,
                                 ScatterMore more, hipStream_t st) {
  if (b.nscatter <= 0) return hipSuccess;
  const hipError_t e =
      scatter_amps(b, win.gamma, mudot, g.dt * g.inv_dx * g.inv_dx * g.inv_dx, st);
  if (e != hipSuccess) return e;
  more.flux = more.flux && more.fp.on && more.fp.nblocks > 0;
  more.sblocks = source_blocks(g, more.src);
  const int nmore = (more.flux ? more.fp.nblocks : 0) + more.src.count * more.sblocks;
  const dim3 grid(b.nscatter + nmore), block(kThreads);
  if (nmore > 0 && b.amp)
    hipLaunchKernelGGL((k_scatter_more<T, true>), grid, block, 0, st, f, g, b, win, mudot, more);
  else if (nmore > 0)
    hipLaunchKernelGGL((k_scatter_more<T, false>), grid, block, 0, st, f, g, b, win, mudot, more);
  else if (b.amp)
    hipLaunchKernelGGL((k_scatter_bins<T, true>), grid, block, 0, st, f, g, b, win, mudot);
  else
    hipLaunchKernelGGL((k_scatter_bins<T, false>), grid, block, 0, st, f, g, b, win, mudot);
  return hipGetLastError();
}

hipError_t bin_scatter_f64(const FieldPtrs<double>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<double>& win, const double* mudot,
                           const ScatterMore& more, hipStream_t st) {
  return launch_scatter<double>(f, g, b, win, mudot, more, st);
}
hipError_t bin_scatter_f32(const FieldPtrs<float>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<float>& win, const double* mudot,
                           const ScatterMore& more, hipStream_t st) {
  return launch_scatter<float>(f, g, b, win, mudot, more, st);
}

template <typename T>
static hipError_t launch_scatter_batch(const ScatterJob<T>* jobs, const int* start, int njobs,
                                       const int2* order, int nblocks, bool amps, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  if (amps)
    hipLaunchKernelGGL((k_scatter_batch<T, true>), dim3(nblocks), dim3(kThreads), 0, st, jobs, start,
                       njobs, order);
  else
    hipLaunchKernelGGL((k_scatter_batch<T, false>), dim3(nblocks), dim3(kThreads), 0, st, jobs, start,
                       njobs, order);
  return hipGetLastError();
}

hipError_t scatter_batch_f64(const ScatterJob<double>* jobs, const int* start, int njobs,
                             const int2* order, int nblocks, bool amps, hipStream_t st) {
  return launch_scatter_batch<double>(jobs, start, njobs, order, nblocks, amps, st);
}
hipError_t scatter_batch_f32(const ScatterJob<float>* jobs, const int* start, int njobs,
                             const int2* order, int nblocks, bool amps, hipStream_t st) {
  return launch_scatter_batch<float>(jobs, start, njobs, order, nblocks, amps, st);
}
hipError_t tls_batch(const TlsJob* jobs, const int* start, int njobs, int nblocks,
                     hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tls_batch, dim3(nblocks), dim3(256), 0, st, jobs, start, njobs);
  return hipGetLastError();
}

// ---- adjoint-step variants
template <typename T, bool AMPS>
__global__ __launch_bounds__(kThreads, ScatterCfg<T>::waves) void k_scatter_plain(
    FieldPtrs<T> f, Geom g, BinPtrs bins, WindowPtrs<T> win, const double* amp, double amp0) {
  scatter_body<T, AMPS, false>(f, g, bins, win, amp, amp0, blockIdx.x);
}
template <typename T>
static hipError_t launch_scatter_plain(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                                       const WindowPtrs<T>& win, const double* amp, double amp0,
                                       hipStream_t st) {
  if (b.nscatter <= 0) return hipSuccess;
  const hipError_t e = scatter_amps(b, win.gamma, amp, amp0, st);
  if (e != hipSuccess) return e;
  if (b.amp)
    hipLaunchKernelGGL((k_scatter_plain<T, true>), dim3(b.nscatter), dim3(kThreads), 0, st, f, g, b,
                       win, amp, amp0);
  else
    hipLaunchKernelGGL((k_scatter_plain<T, false>), dim3(b.nscatter), dim3(kThreads), 0, st, f, g, b,
                       win, amp, amp0);
  return hipGetLastError();
}
hipError_t scatter_plain_f64(const FieldPtrs<double>& f, const Geom& g, const BinPtrs& b,
                             const WindowPtrs<double>& win, const double* amp, double amp0,
                             hipStream_t st) {
  return launch_scatter_plain<double>(f, g, b, win, amp, amp0, st);
}
hipError_t scatter_plain_f32(const FieldPtrs<float>& f, const Geom& g, const BinPtrs& b,
                             const WindowPtrs<float>& win, const double* amp, double amp0,
                             hipStream_t st) {
  return launch_scatter_plain<float>(f, g, b, win, amp, amp0, st);
}

}  // namespace mlk
