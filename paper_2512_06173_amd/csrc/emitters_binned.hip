// Two-level steps and current scatter of the binned emitter phase (the gather is in
// gather.hip).
//
// step (eq. von-Neumann-tls, eq. dipole_derivative): one thread per two-level
// emitter advances its state with the exact propagator and writes mu_dot.
//
// scatter (eqs. J_mol, Polarization_mol):  E_c(p) -= (dt/eps_r(p)) gamma mu_dot^c
// w^c_{m,p} / dx^3.  A workgroup owns a bin of cells and takes every (emitter,
// bin) pair whose window touches the bin, eight lanes per pair; the pair
// carries its window's runs inside the bin, set up on the host.  Contributions
// are summed in LDS (as fixed-point integers, see scatter_body) and each cell
// is written once by its owner (no global atomics).  The pairs' records are
// copied into LDS with 16-byte loads, so the inner loops touch LDS only.
//
// Window weights are the separable factors wx wy wz set up by k_windows, kept
// per emitter as a union-window record (WinRec); a component uses the
// half-integer variant on its own axis.
#include "launch.h"

namespace mlk {

// Scatter bins: 48 KB of accumulators.
template <typename T>
struct BinCfg;
template <>
struct BinCfg<float> {
  static constexpr int SX = 16, SY = 16, SZ = 16;
};
template <>
struct BinCfg<double> {
  static constexpr int SX = 16, SY = 16, SZ = 8;
};

void bin_shape(bool fp32, int G[3], int S[3]) {
  gather_bin_shape(fp32, G);
  if (fp32) {
    S[0] = BinCfg<float>::SX; S[1] = BinCfg<float>::SY; S[2] = BinCfg<float>::SZ;
  } else {
    S[0] = BinCfg<double>::SX; S[1] = BinCfg<double>::SY; S[2] = BinCfg<double>::SZ;
  }
}

namespace {

constexpr int kLanesPerEmitter = 8;  // = kMaxWin: one lane per window x offset
constexpr int kThreads = 512;
constexpr int kGroups = kThreads / kLanesPerEmitter;  // emitters in flight per workgroup
__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

}  // namespace

__global__ __launch_bounds__(256) void k_tls_step(TlsPtrs tls, double dt, const double* Et,
                                                  double* mudot, const int64_t* pop_off,
                                                  Series ser, int64_t n) {
  tls_body(tls, dt, Et, mudot, pop_off, ser, n, blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ __launch_bounds__(256) void k_tls_batch(const TlsJob* jobs, const int* start,
                                                   int njobs) {
  const int j = find_job(start, njobs, blockIdx.x);
  const TlsJob J = load_job(jobs, j);
  const int lb = blockIdx.x - start[j];
  if (lb >= J.nblocks) return;
  tls_body(J.tls, J.dt, J.Et, J.mudot, J.pop_off, J.ser, *J.step,
           lb * blockDim.x + threadIdx.x);
}

// Fixed-point accumulator of the scatter: 32-bit for FP32 fields, 64-bit for FP64.
template <typename T>
struct Acc;
template <>
struct Acc<float> {
  using U = unsigned int;
  using S = int;
  static constexpr int BITS = 30;
  // onto the grid by truncation (one conversion); the grid step is 2^-30 of the
  // bin's bound, far below the FP32 rounding of a cell's sum
  __device__ static S round(float v) { return (S)v; }
};
template <>
struct Acc<double> {
  using U = unsigned long long;
  using S = long long;
  static constexpr int BITS = 62;
  __device__ static S round(double v) { return __double2ll_rn(v); }
};

// scatter; see the file comment.  Contributions are rounded to a fixed-point
// grid chosen per bin and summed as integers in LDS: integer addition is exact
// and order-independent, so the result is deterministic.  In FP32 the Ex and Ey
// sums of a cell share one 64-bit integer, Ey 2^32 + Ex: its sum is exact, and
// since each component's sum stays below 2^30 in magnitude, Ex is the low 32 bits
// read as a signed value and Ey the rest (two LDS atomics per cell, not three).  The grid is
// 2^-BITS of a bound on any cell's sum (|amp| times the largest window weight,
// summed over the bin's emitters): 2^-62 for FP64 fields, far below FP64
// rounding; 2^-30 for FP32 fields, at the level of FP32 rounding of a cell's
// sum.  A contribution is formed in the field precision.
// E_c(p) -= [eps_r^-1(p) if EPS] amp0 gamma a^c w^c_p over the windows, with
// a = mudot (the forward current: amp0 = dt / dx^3, EPS) or any other per-emitter
// amplitude (the adjoint step: amp0 = -1, no EPS).
//
// A pair (emitter, bin) comes with its window's runs inside the bin, one per
// axis, set up on the host (see PairDesc): window offsets d0 .. d0+c-1 on the
// bin-local cells l0 .. l0+c-1.  A window that wraps inside one bin (a periodic
// axis no longer than the bin) is split into several pairs.
//
// Blocks from bins.nscatter on (when fp is given) form the flux partials of the plane
// instead, in the accumulators' LDS.
template <typename T, bool EPS = true>
__device__ __forceinline__ void scatter_body(const FieldPtrs<T>& f, const Geom& g,
                                             const BinPtrs& bins, const WindowPtrs<T>& win,
                                             const double* mudot, double amp0, int bid,
                                             const FluxPlane* fp = nullptr) {
  using A = Acc<T>;
  constexpr int BX = BinCfg<T>::SX, BY = BinCfg<T>::SY, BZ = BinCfg<T>::SZ;
  constexpr int CELLS = BX * BY * BZ;
  constexpr int NW = kThreads / 64;
  constexpr int R4 = sizeof(WinRec<T>) / sizeof(int4);       // 16-byte pieces of a record
  constexpr int NP = (kGroups * R4 + kThreads - 1) / kThreads;  // pieces per thread and chunk
  static_assert(BX <= 16 && BY <= 16 && BZ <= 16, "bin-local run starts take four bits");
  // emitter ids of a bin's pairs kept in LDS (beyond: read from HBM); sized so
  // that two workgroups still fit one CU's LDS
  constexpr int kIdCap = sizeof(T) == 4 ? 4096 : 1024;
  __shared__ alignas(16) typename A::U sJ[3][CELLS];
  // FP32: Ex and Ey share one 64-bit accumulator per cell (sJ[0] and sJ[1] reused),
  // two LDS atomics per cell instead of three
  constexpr bool kPackXY = sizeof(T) == 4;
  unsigned long long* const sJxy = reinterpret_cast<unsigned long long*>(&sJ[0][0]);
  __shared__ WinRec<T> sW[kGroups];
  __shared__ T sAmp[kGroups][3];
  __shared__ unsigned sRun[kGroups];
  __shared__ int sId[kIdCap];
  __shared__ double sRed[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (fp && bid >= bins.nscatter) {  // uniform across the block
    flux_partial_sum(f, g, *fp, bid - bins.nscatter, fp->nblocks,
                     reinterpret_cast<double*>(&sJ[0][0]));
    return;
  }
  const int b = bins.sbin_id[bid];
  const int bx = b % bins.nbx, by = (b / bins.nbx) % bins.nby, bz = b / (bins.nbx * bins.nby);
  const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;
  const int ex = min(BX, g.n[0] - x0), ey = min(BY, g.n[1] - y0), ez = min(BZ, g.n[2] - z0);
  const int q0 = bins.sbin_start[bid], q1 = bins.sbin_start[bid + 1];
  {
    // cleared 16 bytes at a time (the three accumulator arrays are contiguous)
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    u4* z = reinterpret_cast<u4*>(&sJ[0][0]);
    constexpr int NZ = 3 * CELLS * (int)sizeof(typename A::U) / 16;
    for (int t = tid; t < NZ; t += kThreads) z[t] = u4{0u, 0u, 0u, 0u};
  }
  double bound = 0.0;
  for (int q = q0 + tid; q < q1; q += kThreads) {
    const int4 pd = bins.sbin_pair[q];
    if (q - q0 < kIdCap) sId[q - q0] = pd.x;
    bound += (double)__int_as_float(pd.z) *
             (fabs(mudot[3 * pd.x]) + fabs(mudot[3 * pd.x + 1]) + fabs(mudot[3 * pd.x + 2]));
  }
  bound = wave_sum64(bound);
  if (lane == 0) sRed[wave] = bound;
  __syncthreads();
  bound = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) bound += sRed[w];
  bound *= fabs(amp0);
  if (!(bound > 0.0)) return;  // nothing to add in this bin (uniform across the block)
  // scale = 2^(BITS - e) with bound < 2^e: every partial sum stays below 2^BITS
  const int ebits = ilogb(bound) + 1;
  const double scale = ldexp(1.0, A::BITS - ebits);
  const double inv_scale = ldexp(1.0, ebits - A::BITS);

  // The pairs are taken in chunks of kGroups.  With FP32 fields the next
  // chunk's window records, runs and amplitudes (gamma, mu_dot) are loaded into
  // registers while the current chunk is summed, and moved to LDS behind an
  // LDS-only barrier, so their HBM latency overlaps the atomics instead of
  // stalling every chunk.  FP64 records are twice as large: holding them across
  // the sums would cost the second workgroup per CU, so FP64 loads each chunk
  // right before storing it.
  constexpr bool kPipe = sizeof(T) == 4;
  typedef int piece_t __attribute__((ext_vector_type(4)));  // kept in registers
  piece_t piece[NP];
  double pg = 0.0, pm0 = 0.0, pm1 = 0.0, pm2 = 0.0;
  unsigned prun = 0;
  // Eight lanes per pair, lane i on the i-th window x offset of the pair's x run;
  // the group walks the cy x cz rows and planes of its y and z runs, so a
  // wavefront runs its eight groups' loops side by side for as many steps as its
  // longest group; the host orders the pairs of a bin by (cz, cy) so that
  // neighbouring groups have equal counts.
  const int grp = tid / kLanesPerEmitter, i = tid % kLanesPerEmitter;
  // loads of the chunk at c: pieces (clamped to the chunk's last record) and, for
  // tid < the chunk size, the runs and amplitude inputs of pair tid
#define MLK_STAGE_LOAD(c)                                                             \
  {                                                                                  \
    const int cl = min(kGroups, q1 - (c)) - 1;                                       \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                 \
      const int idx = tid + p * kThreads, sl = min(idx / R4, cl);                    \
      const int q = (c) + sl;                                                        \
      const int em = q - q0 < kIdCap ? sId[q - q0] : bins.sbin_pair[q].x;            \
      piece[p] = reinterpret_cast<const piece_t*>(win.rec + em)[idx % R4];           \
    }                                                                                \
    const int q = (c) + min(tid, cl);                                                \
    const int4 pd = bins.sbin_pair[q];                                               \
    prun = (unsigned)pd.y;                                                           \
    pg = win.gamma[pd.x];                                                            \
    pm0 = mudot[3 * pd.x];                                                           \
    pm1 = mudot[3 * pd.x + 1];                                                       \
    pm2 = mudot[3 * pd.x + 2];                                                       \
  }
  if (kPipe) MLK_STAGE_LOAD(q0)
  for (int c0 = q0; c0 < q1; c0 += kGroups) {
    const int cn = min(kGroups, q1 - c0);
    if (c0 > q0) lds_barrier();  // the previous chunk's records are no longer read
    if (!kPipe) MLK_STAGE_LOAD(c0)
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int idx = tid + p * kThreads;
      if (idx < cn * R4) reinterpret_cast<piece_t*>(sW + idx / R4)[idx % R4] = piece[p];
    }
    if (tid < cn) {
      const double ge = amp0 * pg * scale;
      sAmp[tid][0] = (T)(ge * pm0);
      sAmp[tid][1] = (T)(ge * pm1);
      sAmp[tid][2] = (T)(ge * pm2);
      sRun[tid] = prun;
    }
    lds_barrier();
    if (kPipe && c0 + kGroups < q1) MLK_STAGE_LOAD(c0 + kGroups)
    if (grp >= cn) continue;
    const unsigned run = sRun[grp];
    const int nx = ((run >> 7) & 7) + 1;
    if (i >= nx) continue;
    const WinRec<T>& w = sW[grp];
    const int li = (run & 15) + i, dxi = ((run >> 4) & 7) + i;
    const int ly0 = (run >> 10) & 15, dy0 = (run >> 14) & 7, cj = ((run >> 17) & 7) + 1;
    const int lz0 = (run >> 20) & 15, dz0 = (run >> 24) & 7, ck = ((run >> 27) & 7) + 1;
    T wy0[kMaxWin], wy1[kMaxWin], wz0[kMaxWin], wz1[kMaxWin];
#pragma unroll
    for (int r = 0; r < kMaxWin; ++r) {
      // offsets past the run are clamped into the record and never used
      const int dy = min(dy0 + r, kMaxWin - 1), dz = min(dz0 + r, kMaxWin - 1);
      wy0[r] = w.wr[1][0][dy];
      wy1[r] = w.wr[1][1][dy];
      wz0[r] = w.wr[2][0][dz];
      wz1[r] = w.wr[2][1][dz];
    }
    const T cx = sAmp[grp][0] * w.wr[0][1][dxi];
    const T cy = sAmp[grp][1] * w.wr[0][0][dxi];
    const T cz = sAmp[grp][2] * w.wr[0][0][dxi];
    const int base = BX * (ly0 + BY * lz0) + li;
#pragma unroll
    for (int k = 0; k < kMaxWin; ++k) {
      if (k >= ck) break;
      const T cxk = cx * wz0[k], cyk = cy * wz0[k], czk = cz * wz1[k];
      const int pk = base + BX * BY * k;
#pragma unroll
      for (int j = 0; j < kMaxWin; ++j) {
        if (j >= cj) break;
        const int s = pk + BX * j;
        if constexpr (kPackXY) {
          // Ex and Ey in one 64-bit integer, Ey 2^32 + Ex (both sums stay below 2^30)
          const long long pxy = (long long)A::round(cyk * wy1[j]) * 4294967296LL +
                                (long long)A::round(cxk * wy0[j]);
          atomicAdd(sJxy + s, (unsigned long long)pxy);
        } else {
          atomicAdd(&sJ[0][s], (typename A::U)A::round(cxk * wy0[j]));
          atomicAdd(&sJ[1][s], (typename A::U)A::round(cyk * wy1[j]));
        }
        atomicAdd(&sJ[2][s], (typename A::U)A::round(czk * wy0[j]));
      }
    }
  }
#undef MLK_STAGE_LOAD
  __syncthreads();
  // owner write: E -= [eps^-1] J on the cells of this bin; the loads of a thread's
  // cells are issued together (unconditional, from a safe index: cell 0 for a
  // cell that no window reaches, so only touched cells cost HBM reads), then the
  // stores
  static_assert(CELLS % kThreads == 0, "the bin is a whole number of workgroup passes");
  constexpr int RW = CELLS / kThreads;
  typename A::S jv[RW][3];
  size_t idw[RW];
  T ev[RW][3], eiv[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int t = tid + r * kThreads;
    const int li = t % BX, lj = (t / BX) % BY, lk = t / (BX * BY);
    const bool in = li < ex && lj < ey && lk < ez;
#pragma unroll
    for (int c = 0; c < 3; ++c) jv[r][c] = in ? (typename A::S)sJ[c][t] : 0;
    if constexpr (kPackXY) {
      // the packed sum is Ey 2^32 + Ex exactly; |Ex| < 2^31, so Ex is its low 32 bits
      // read as a signed value, and Ey what remains
      const long long pxy = in ? (long long)sJxy[t] : 0LL;
      const int lx = (int)(unsigned)(unsigned long long)pxy;
      jv[r][0] = lx;
      jv[r][1] = (typename A::S)((pxy - (long long)lx) / 4294967296LL);
    }
    const bool hit = in && (jv[r][0] | jv[r][1] | jv[r][2]) != 0;
    idw[r] = hit ? cell_index(g, x0 + li, y0 + lj, z0 + lk) : 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) ev[r][c] = f.E[c][idw[r]];
    eiv[r] = (EPS && f.epsinv) ? f.epsinv[idw[r]] : T(1);  // null: eps_r = 1 everywhere
  }
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (jv[r][c] != 0) f.E[c][idw[r]] = ev[r][c] - eiv[r] * (T)((double)jv[r][c] * inv_scale);
}

template <typename T>
__global__ __launch_bounds__(kThreads, 4) void k_scatter_bins(FieldPtrs<T> f, Geom g, BinPtrs bins,
                                                           WindowPtrs<T> win,
                                                           const double* mudot) {
  scatter_body(f, g, bins, win, mudot, g.dt * g.inv_dx * g.inv_dx * g.inv_dx, blockIdx.x);
}

// The scatter with the flux partials of the plane in fp.nblocks more workgroups.
template <typename T>
__global__ __launch_bounds__(kThreads, 4) void k_scatter_flux(FieldPtrs<T> f, Geom g, BinPtrs bins,
                                                           WindowPtrs<T> win,
                                                           const double* mudot, FluxPlane fp) {
  scatter_body(f, g, bins, win, mudot, g.dt * g.inv_dx * g.inv_dx * g.inv_dx, blockIdx.x, &fp);
}

template <typename T>
__global__ __launch_bounds__(kThreads, 4) void k_scatter_batch(const ScatterJob<T>* jobs,
                                                            const int* start, int njobs,
                                                            const int2* order) {
  int j, bid;
  if (order) {  // (job, bin) of the block, heaviest first across the jobs
    const int2 o = order[blockIdx.x];
    j = o.x;
    bid = o.y;
  } else {
    j = find_job(start, njobs, blockIdx.x);
    bid = blockIdx.x - start[j];
    if (bid >= jobs[j].nblocks) return;
  }
  const ScatterJob<T> J = load_job(jobs, j);
  scatter_body(J.f, J.g, J.bins, J.win, J.mudot, J.g.dt * J.g.inv_dx * J.g.inv_dx * J.g.inv_dx,
               bid);
}

hipError_t tls_step(const TlsPtrs& tls, double dt, const double* Et, double* mudot,
                    const int64_t* pop_off, const Series& ser, int64_t n, hipStream_t st) {
  if (tls.count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tls_step, dim3((tls.count + 255) / 256), dim3(256), 0, st, tls, dt, Et,
                     mudot, pop_off, ser, n);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_scatter(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                                 const WindowPtrs<T>& win, const double* mudot,
                                 const FluxPlane* fp, hipStream_t st) {
  if (b.nscatter <= 0) return hipSuccess;
  if (fp && fp->on && fp->nblocks > 0)
    hipLaunchKernelGGL(k_scatter_flux<T>, dim3(b.nscatter + fp->nblocks), dim3(kThreads), 0, st,
                       f, g, b, win, mudot, *fp);
  else
    hipLaunchKernelGGL(k_scatter_bins<T>, dim3(b.nscatter), dim3(kThreads), 0, st, f, g, b, win,
                       mudot);
  return hipGetLastError();
}

hipError_t bin_scatter_f64(const FieldPtrs<double>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<double>& win, const double* mudot,
                           const FluxPlane* fp, hipStream_t st) {
  return launch_scatter<double>(f, g, b, win, mudot, fp, st);
}
hipError_t bin_scatter_f32(const FieldPtrs<float>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<float>& win, const double* mudot,
                           const FluxPlane* fp, hipStream_t st) {
  return launch_scatter<float>(f, g, b, win, mudot, fp, st);
}

template <typename T>
static hipError_t launch_scatter_batch(const ScatterJob<T>* jobs, const int* start, int njobs,
                                       const int2* order, int nblocks, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_batch<T>, dim3(nblocks), dim3(kThreads), 0, st, jobs, start, njobs,
                     order);
  return hipGetLastError();
}

hipError_t scatter_batch_f64(const ScatterJob<double>* jobs, const int* start, int njobs,
                             const int2* order, int nblocks, hipStream_t st) {
  return launch_scatter_batch<double>(jobs, start, njobs, order, nblocks, st);
}
hipError_t scatter_batch_f32(const ScatterJob<float>* jobs, const int* start, int njobs,
                             const int2* order, int nblocks, hipStream_t st) {
  return launch_scatter_batch<float>(jobs, start, njobs, order, nblocks, st);
}
hipError_t tls_batch(const TlsJob* jobs, const int* start, int njobs, int nblocks,
                     hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tls_batch, dim3(nblocks), dim3(256), 0, st, jobs, start, njobs);
  return hipGetLastError();
}

// ---- adjoint-step variants
template <typename T>
__global__ __launch_bounds__(kThreads, 4) void k_scatter_plain(FieldPtrs<T> f, Geom g, BinPtrs bins,
                                                            WindowPtrs<T> win, const double* amp,
                                                            double amp0) {
  scatter_body<T, false>(f, g, bins, win, amp, amp0, blockIdx.x);
}
template <typename T>
static hipError_t launch_scatter_plain(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                                       const WindowPtrs<T>& win, const double* amp, double amp0,
                                       hipStream_t st) {
  if (b.nscatter <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_plain<T>, dim3(b.nscatter), dim3(kThreads), 0, st, f, g, b, win,
                     amp, amp0);
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
