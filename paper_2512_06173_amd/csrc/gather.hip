// Field gather of the emitters (eq. E_regu_Emi): E~_m = gamma_m sum_p w_{m,p} E(p).
//
// The emitters are grouped by the bin of their centre cell.  The workgroup of a bin
// stages E over the bin plus the windows' reach in LDS, which holds every window of
// its emitters.  Eight lanes (FP32 fields) or sixteen (FP64) serve one emitter, lane
// (i, h) taking the x offset i of its window and the h-th share of its rows: a lane
// sums its rows along y in the field precision, weights them along z into FP64, and
// the lanes of the emitter add up their sums (FP64).
//
// The tile goes from memory to LDS directly (global_load_lds, 16 bytes a lane where
// rows allow it), without passing through registers: a few instructions a thread
// instead of eighteen loads, and the emitter's record is fetched into registers while
// the tile is on its way instead of after it.  The tile reaches as far as the
// windows do (three cells for R sigma <= 3, else four; x stays four, a 16-byte
// boundary): 24 x 14 x 14 cells in FP32, 56 KB, and 16 x 14 x 14 in FP64, 75 KB, so two
// workgroups share a CU in both.
//
// Bins are handed out XCD by XCD so that neighbouring bins, whose tiles overlap,
// share one L2.  Bins of few emitters ("light") need no tile: a wavefront per emitter
// reads its window from memory, in workgroups behind those of the tiled bins; behind
// those, more workgroups save the flux plane's E^n.
//
// The emitters' window weights are the separable factors wx wy wz of their
// union-window records (WinRec); a component uses the half-integer variant on its own
// axis.
#include "launch.h"

namespace mlk {

namespace {

constexpr int kLanesPerEmitter = 8;  // = kMaxWin: one lane per window x offset

// Tile and launch shape.  R: reach of the windows along y and z (3 or 4 cells).  WEPS:
// 1/eps_r is staged beside E (the adjoint's gather of eps_r^-1 E).  An emitter takes
// `lanes` lanes, lane (i, h) on window x offset i and rows h*rows .. h*rows+rows-1.
// FP64 splits the rows over sixteen lanes, which halves the chain of each lane's sums
// and its registers; FP32 is faster with eight (52.7 us against 55.6 when measured).
template <typename T, int R, bool WEPS>
struct GatherCfg {
  static constexpr int BX = sizeof(T) == 4 ? 16 : 8, BY = 8, BZ = 8;
  static constexpr int TX = BX + 2 * kHalo, TY = BY + 2 * R, TZ = BZ + 2 * R;
  static constexpr int cells = TX * TY * TZ, arrays = WEPS ? 4 : 3;
  static constexpr bool two = 2 * arrays * cells * sizeof(T) <= 160 * 1024;  // per CU
  static constexpr int threads = (sizeof(T) == 8 || WEPS) && two ? 512 : 1024;
  static constexpr int waves_per_simd = threads / 256 * (two ? 2 : 1);
  static constexpr int lanes = sizeof(T) == 4 ? 8 : 16;
  static constexpr int rows = kMaxWin * kLanesPerEmitter / lanes;
};

// sum over the L consecutive lanes of one gather emitter
template <int L>
__device__ __forceinline__ double gather_lane_sum(double v) {
#pragma unroll
  for (int off = L / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, L);
  return v;
}

// One plane's term of an emitter's z sum, a + wz s, rounded alike by every gather
// path: in FP64 as one fused multiply-add, in FP32 with the product rounded in FP32
// and the sum in FP64.
__device__ __forceinline__ double zterm(double a, double wz, double s) {
  return __builtin_fma(wz, s, a);
}
__device__ __forceinline__ double zterm(double a, float wz, float s) {
  return a + (double)(wz * s);
}

// Index q of an axis as the tile reads it: wrapped on a periodic axis, else held
// inside the grid (no window reaches beyond a wall, so what such a slot holds is
// never used).
__device__ __forceinline__ int tile_index(int q, int n, int last, int periodic) {
  if (!periodic) return min(max(q, 0), last);
  const int m = q % n;
  return m < 0 ? m + n : m;
}

// U bytes a lane from src to LDS, the lanes' units one after another from dst (uniform).
template <int U>
__device__ __forceinline__ void load_to_lds(const char* src, char* dst) {
  const auto* s = (const __attribute__((address_space(1))) void*)src;
  auto* d = (__attribute__((address_space(3))) void*)dst;
  if constexpr (U == 16) __builtin_amdgcn_global_load_lds(s, d, 16, 0, 0);
  else __builtin_amdgcn_global_load_lds(s, d, 4, 0, 0);
}

// The tile of the box whose low corner is (x0, y0, z0) from memory to LDS, U bytes a
// lane and array.  LDS takes a wavefront's units one after another from a uniform
// base, so unit u of the tile (rows of TX cells, one after another) sits at byte U u.
template <typename T, int R, bool WEPS, int U>
__device__ __forceinline__ void fill_tile(const FieldPtrs<T>& f, const Geom& g, int x0, int y0,
                                          int z0, T* lds) {
  using C = GatherCfg<T, R, WEPS>;
  constexpr int UR = C::TX * (int)sizeof(T) / U, NU = UR * C::TY * C::TZ;
  constexpr int UE = U > (int)sizeof(T) ? U / (int)sizeof(T) : 1;  // cells a unit holds
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int u0 = wave * 64; u0 < NU; u0 += C::threads) {
    const int u = u0 + lane;
    if (u >= NU) break;
    const int row = u / UR, b = (u % UR) * U;
    const int i = tile_index(x0 + b / (int)sizeof(T), g.n[0], g.n[0] - UE, g.periodic[0]);
    const int j = tile_index(y0 + row % C::TY, g.n[1], g.n[1] - 1, g.periodic[1]);
    const int k = tile_index(z0 + row / C::TY, g.n[2], g.n[2] - 1, g.periodic[2]);
    const size_t at = cell_index(g, i, j, k) * sizeof(T) + b % sizeof(T);
#pragma unroll
    for (int c = 0; c < C::arrays; ++c) {
      const char* src = reinterpret_cast<const char*>(c < 3 ? f.E[c < 3 ? c : 0] : f.epsinv) + at;
      char* dst = reinterpret_cast<char*>(lds + c * C::cells) + u0 * U;
      load_to_lds<U>(src, dst);
    }
  }
}

// The part of an emitter's window record that one gather lane needs, in registers:
// where its window starts in the tile, the lane's own x weights, the y weights of its
// rows and every z weight (the lanes of an emitter read the same record).
template <typename T, int ROWS>
struct LaneWin {
  int base, nx, ny, nz;  // tile index of the lane's first cell; extents (ny: its rows)
  T wx0, wx1;
  T wy[2][ROWS], wz[2][kMaxWin];
};

template <typename T, int R, bool WEPS, int ROWS>
__device__ __forceinline__ void load_lane_win(const WinRec<T>& r, int i, int j0, int x0, int y0,
                                              int z0, LaneWin<T, ROWS>& w) {
  using C = GatherCfg<T, R, WEPS>;
  const int4 o = *reinterpret_cast<const int4*>(&r.org[0]);  // org[0..2], n[0]
  const int2 nn = *reinterpret_cast<const int2*>(&r.n[1]);
  w.base = (o.x + i - x0) + C::TX * (o.y + j0 - y0) + C::TX * C::TY * (o.z - z0);
  w.nx = o.w;
  w.ny = nn.x - j0;
  w.nz = nn.y;
  w.wx0 = r.wr[0][i][0];
  w.wx1 = r.wr[0][i][1];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
#pragma unroll
    for (int d = 0; d < ROWS; ++d) w.wy[v][d] = r.wr[1][j0 + d][v];
#pragma unroll
    for (int d = 0; d < kMaxWin; ++d) w.wz[v][d] = r.wr[2][d][v];
  }
}

template <typename T, int R, bool WEPS, int U>
__device__ __forceinline__ void tile_body(const FieldPtrs<T>& f, const Geom& g,
                                          const BinPtrs& bins, const WindowPtrs<T>& win,
                                          double* Et, int bid) {
  using C = GatherCfg<T, R, WEPS>;
  constexpr int LG = C::lanes, NG = C::threads / LG, RG = C::rows;
  __shared__ alignas(16) T sE[C::arrays * C::cells];
  const int tid = threadIdx.x;
  const int bin = xcd_block(bid, bins.gdense);
  // tile origin in the unwrapped frame of the emitters' window indices
  const int x0 = bins.gbin_org[3 * bin] - kHalo;
  const int y0 = bins.gbin_org[3 * bin + 1] - R;
  const int z0 = bins.gbin_org[3 * bin + 2] - R;
  fill_tile<T, R, WEPS, U>(f, g, x0, y0, z0, sE);
  // the first emitter's record is fetched while the tile is on its way
  const int grp = tid / LG, i = tid % kLanesPerEmitter;
  const int j0 = (tid / kLanesPerEmitter) % (LG / kLanesPerEmitter) * RG;
  const int q0 = bins.gbin_start[bin], q1 = bins.gbin_start[bin + 1];
  int e = 0;
  LaneWin<T, RG> w;
  if (q0 + grp < q1) {
    e = bins.gbin_em[q0 + grp];
    load_lane_win<T, R, WEPS, RG>(win.rec[q0 + grp], i, j0, x0, y0, z0, w);
  }
  // every wavefront waits for its own units, the barrier for those of the others
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  for (int q = q0 + grp; q < q1;) {  // uniform across the lanes of an emitter
    double ax = 0.0, ay = 0.0, az = 0.0;
    if (i < w.nx) {
      // The sums read every row of a plane before adding them up (no branch per
      // row), one component at a time, so that the reads of a plane are in flight
      // together.  Rows past the window (j >= ny) read the window's first row, a
      // staged cell, with the record's zero weight: their terms are zeros and leave
      // the sums as they are.
      int roff[RG];
#pragma unroll
      for (int j = 0; j < RG; ++j) roff[j] = j < w.ny ? C::TX * j : -C::TX * j0;
      // Ex and Ez take the integer y weights, Ey the half-integer ones; Ez the
      // half-integer z weights
      auto comp = [&](int c, const T* wy, const T* wz) -> double {
        double a = 0.0;
        int sk = w.base;
#pragma unroll
        for (int k = 0; k < kMaxWin; ++k, sk += C::TX * C::TY) {
          if (k < w.nz) {
            T v[RG];
#pragma unroll
            for (int j = 0; j < RG; ++j) {
              v[j] = sE[c * C::cells + sk + roff[j]];
              if (WEPS) v[j] *= sE[(C::arrays - 1) * C::cells + sk + roff[j]];
            }
            T sc = T(0);
#pragma unroll
            for (int j = 0; j < RG; ++j) sc += wy[j] * v[j];
            a = zterm(a, wz[k], sc);
          }
        }
        return a;
      };
      ax = comp(0, w.wy[0], w.wz[0]);
      ay = comp(1, w.wy[1], w.wz[0]);
      az = comp(2, w.wy[0], w.wz[1]);
      // Ex sits at half-integer x (variant 1); Ey, Ez at integer x
      ax *= (double)w.wx1;
      ay *= (double)w.wx0;
      az *= (double)w.wx0;
    }
    ax = gather_lane_sum<LG>(ax);
    ay = gather_lane_sum<LG>(ay);
    az = gather_lane_sum<LG>(az);
    if (tid % LG == 0) {
      const double gm = win.gamma[e];
      Et[3 * e] = gm * ax;
      Et[3 * e + 1] = gm * ay;
      Et[3 * e + 2] = gm * az;
    }
    q += NG;
    if (q < q1) {
      e = bins.gbin_em[q];
      load_lane_win<T, R, WEPS, RG>(win.rec[q], i, j0, x0, y0, z0, w);
    }
  }
}

// The q-th emitter of the light bins, without a tile, by one wavefront: lane (i, k) on
// window x offset i and plane k, reading its window cells from memory (every row of
// its plane, for each of the row groups h that the tiled gather gives separate
// lanes).  A lane forms the tiled gather's row sums sum_j wy E for its plane; the
// plane-0 lanes then take the z sums in plane order, scale by the x weight, join the
// row groups and sum over x as the tiled gather's lanes do, so E~ is the same bit for
// bit.  All planes' loads are in flight together.  The emitter is the same for the
// whole wavefront, so its record comes through scalar loads.
template <typename T, bool WEPS>
__device__ __forceinline__ void light_body(const FieldPtrs<T>& f, const Geom& g,
                                           const BinPtrs& bins, const WindowPtrs<T>& win,
                                           double* Et, int q) {
  using C = GatherCfg<T, 3, false>;
  constexpr int RG = C::rows, H = C::lanes / kLanesPerEmitter;
  static_assert(kLanesPerEmitter * kMaxWin == 64, "one lane per (x offset, plane)");
  const int lane = threadIdx.x & 63;
  const int i = lane % kLanesPerEmitter, k = lane / kLanesPerEmitter;
  const int em = __builtin_amdgcn_readfirstlane(bins.glight0 + q);
  const int e = __builtin_amdgcn_readfirstlane(bins.gbin_em[em]);
#if defined(__HIP_DEVICE_COMPILE__)
  const auto& r = ((__attribute__((address_space(4))) const WinRec<T>*)win.rec)[em];
#else
  const auto& r = win.rec[em];
#endif
  const int nx = r.n[0], nyw = r.n[1], nz = r.n[2];
  T t[H][3];  // the lane's row sums of its plane, per row group and component
#pragma unroll
  for (int h = 0; h < H; ++h) t[h][0] = t[h][1] = t[h][2] = T(0);
  if (i < nx && k < nz) {
    // (no window reaches beyond a wall; wrapped on a periodic axis)
    const int cx = tile_index(r.org[0] + i, g.n[0], g.n[0] - 1, g.periodic[0]);
    const int cz = tile_index(r.org[2] + k, g.n[2], g.n[2] - 1, g.periodic[2]);
    T v[H][RG][3];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int j = 0; j < RG; ++j) {
        // rows past the window read its first row, with the record's zero weight
        const int d = h * RG + j < nyw ? h * RG + j : 0;
        const int cy = tile_index(r.org[1] + d, g.n[1], g.n[1] - 1, g.periodic[1]);
        const size_t id = cell_index(g, cx, cy, cz);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[h][j][c] = f.E[c][id];
        if (WEPS) {
          const T ei = f.epsinv[id];
#pragma unroll
          for (int c = 0; c < 3; ++c) v[h][j][c] *= ei;
        }
      }
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int j = 0; j < RG; ++j) {
        const T wy0 = r.wr[1][h * RG + j][0], wy1 = r.wr[1][h * RG + j][1];
        t[h][0] += wy0 * v[h][j][0];
        t[h][1] += wy1 * v[h][j][1];
        t[h][2] += wy0 * v[h][j][2];
      }
  }
  // the z sums in plane order (every lane takes part in the shuffles; the plane-0
  // lanes keep the sums); Ez takes the half-integer z weights
  double a[H][3];
#pragma unroll
  for (int h = 0; h < H; ++h) a[h][0] = a[h][1] = a[h][2] = 0.0;
#pragma unroll
  for (int kk = 0; kk < kMaxWin; ++kk) {
    if (kk < nz) {  // uniform across the wavefront
      const T wz0 = r.wr[2][kk][0], wz1 = r.wr[2][kk][1];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int src = i + kLanesPerEmitter * kk;
        a[h][0] = zterm(a[h][0], wz0, __shfl(t[h][0], src, 64));
        a[h][1] = zterm(a[h][1], wz0, __shfl(t[h][1], src, 64));
        a[h][2] = zterm(a[h][2], wz1, __shfl(t[h][2], src, 64));
      }
    }
  }
  if (i < nx) {
    // Ex sits at half-integer x (variant 1); Ey, Ez at integer x
    const double wx0 = (double)win.rec[em].wr[0][i][0], wx1 = (double)win.rec[em].wr[0][i][1];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      a[h][0] *= wx1;
      a[h][1] *= wx0;
      a[h][2] *= wx0;
    }
  }
  // the row groups of one x offset, then the x offsets: the tiled gather's lane sum
  double ax = a[0][0], ay = a[0][1], az = a[0][2];
  if (H == 2) {
    ax += a[H - 1][0];
    ay += a[H - 1][1];
    az += a[H - 1][2];
  }
  ax = gather_lane_sum<kLanesPerEmitter>(ax);
  ay = gather_lane_sum<kLanesPerEmitter>(ay);
  az = gather_lane_sum<kLanesPerEmitter>(az);
  if (lane == 0) {
    const double gm = win.gamma[e];
    Et[3 * e] = gm * ax;
    Et[3 * e + 1] = gm * ay;
    Et[3 * e + 2] = gm * az;
  }
}

// Workgroup b of a gather: tiled bins, then the light bins' emitters, a wavefront each.
template <typename T, int R, bool WEPS, int U>
__device__ __forceinline__ void gather_body(const FieldPtrs<T>& f, const Geom& g,
                                            const BinPtrs& bins, const WindowPtrs<T>& win,
                                            double* Et, int b) {
  constexpr int W = GatherCfg<T, R, WEPS>::threads / 64;
  if (b < bins.gdense) {  // uniform across the workgroup
    tile_body<T, R, WEPS, U>(f, g, bins, win, Et, b);
    return;
  }
  const int q = (b - bins.gdense) * W + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (q < bins.nlight) light_body<T, WEPS>(f, g, bins, win, Et, q);
}

}  // namespace

template <typename T, int R, bool WEPS, int U>
__global__ __launch_bounds__((GatherCfg<T, R, WEPS>::threads),
                             (GatherCfg<T, R, WEPS>::waves_per_simd))
void k_gather(FieldPtrs<T> f, Geom g, BinPtrs bins, WindowPtrs<T> win, double* Et, int nblocks,
              FluxPlane fp) {
  if ((int)blockIdx.x >= nblocks) {  // uniform across the workgroup
    flux_save_body(f, g, fp, ((int)blockIdx.x - nblocks) * GatherCfg<T, R, WEPS>::threads +
                                 (int)threadIdx.x);
    return;
  }
  gather_body<T, R, WEPS, U>(f, g, bins, win, Et, blockIdx.x);
}

template <typename T, int R, int U>
__global__ __launch_bounds__((GatherCfg<T, R, false>::threads),
                             (GatherCfg<T, R, false>::waves_per_simd))
void k_gather_batch(const GatherJob<T>* jobs, const int2* order) {
  const int2 o = order[blockIdx.x];  // (job, workgroup), heaviest first across the jobs
  const GatherJob<T> J = load_job(jobs, o.x);
  gather_body<T, R, false, U>(J.f, J.g, J.bins, J.win, J.Et, o.y);
}

namespace {

template <typename T>
int gather_threads(int reach) {
  return reach <= 3 ? GatherCfg<T, 3, false>::threads : GatherCfg<T, 4, false>::threads;
}

// 16-byte units need rows and arrays on 16-byte boundaries; else 4-byte units.
template <typename T>
bool wide_units(const FieldPtrs<T>& f, const Geom& g, bool weps) {
  bool ok = (size_t)g.n[0] * sizeof(T) % 16 == 0;
  for (int c = 0; c < 3; ++c) ok = ok && ((uintptr_t)f.E[c] & 15) == 0;
  return ok && (!weps || ((uintptr_t)f.epsinv & 15) == 0);
}

template <typename T, int R, bool WEPS, int U>
hipError_t launch_gather_t(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<T>& win, double* Et, const FluxPlane* fp,
                           hipStream_t st) {
  constexpr int NT = GatherCfg<T, R, WEPS>::threads;
  int nflux = 0;
  FluxPlane fpv{};
  if (fp) {
    const int a = fp->axis, u = (a + 1) % 3, v = (a + 2) % 3;
    nflux = (g.n[u] * g.n[v] + NT - 1) / NT;
    fpv = *fp;
  }
  const int nblocks = b.gdense + (b.nlight + NT / 64 - 1) / (NT / 64);
  if (nblocks + nflux == 0) return hipSuccess;
  hipLaunchKernelGGL((k_gather<T, R, WEPS, U>), dim3(nblocks + nflux), dim3(NT), 0, st, f, g, b,
                     win, Et, nblocks, fpv);
  return hipGetLastError();
}

template <typename T, bool WEPS>
hipError_t launch_gather(const FieldPtrs<T>& f, const Geom& g, const BinPtrs& b,
                         const WindowPtrs<T>& win, double* Et, const FluxPlane* fp,
                         hipStream_t st) {
  if (b.ngather <= 0) return fp ? hipErrorInvalidValue : hipSuccess;
  const bool wide = wide_units(f, g, WEPS);
  if (b.reach <= 3)
    return wide ? launch_gather_t<T, 3, WEPS, 16>(f, g, b, win, Et, fp, st)
                : launch_gather_t<T, 3, WEPS, 4>(f, g, b, win, Et, fp, st);
  return wide ? launch_gather_t<T, 4, WEPS, 16>(f, g, b, win, Et, fp, st)
              : launch_gather_t<T, 4, WEPS, 4>(f, g, b, win, Et, fp, st);
}

template <typename T>
hipError_t launch_gather_batch(const GatherJob<T>* jobs, const int2* order, int nblocks, int reach,
                               bool wide, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  const dim3 grid(nblocks), block(gather_threads<T>(reach));
  if (reach <= 3 && wide)
    hipLaunchKernelGGL((k_gather_batch<T, 3, 16>), grid, block, 0, st, jobs, order);
  else if (reach <= 3)
    hipLaunchKernelGGL((k_gather_batch<T, 3, 4>), grid, block, 0, st, jobs, order);
  else if (wide)
    hipLaunchKernelGGL((k_gather_batch<T, 4, 16>), grid, block, 0, st, jobs, order);
  else
    hipLaunchKernelGGL((k_gather_batch<T, 4, 4>), grid, block, 0, st, jobs, order);
  return hipGetLastError();
}

}  // namespace

void gather_bin_shape(bool fp32, int G[3]) {
  using F = GatherCfg<float, 3, false>;
  using D = GatherCfg<double, 3, false>;
  G[0] = fp32 ? F::BX : D::BX;
  G[1] = fp32 ? F::BY : D::BY;
  G[2] = fp32 ? F::BZ : D::BZ;
}

// A bin of at most this many emitters is light: a wavefront reads 8^3 cells per
// emitter, a workgroup 14 x 14 rows for all of them.  Step times with 2, 4, 8 and 16:
// 160^3 with 10,000 emitters 149.7, 148.1, 143.8, 142.2 us; 187 x 149 x 163 FP64 with
// 20,000 311, 299, 293, 295; 384^3 with 100,000 949, 950, 949, 963; 64-domain batch 585,
// 576, 575, 577.
int gather_light_max() { return 8; }

int gather_light_blocks(bool fp32, int reach, int nlight) {
  const int w = (fp32 ? gather_threads<float>(reach) : gather_threads<double>(reach)) / 64;
  return (nlight + w - 1) / w;
}

bool gather_wide_f64(const FieldPtrs<double>& f, const Geom& g) { return wide_units(f, g, false); }
bool gather_wide_f32(const FieldPtrs<float>& f, const Geom& g) { return wide_units(f, g, false); }

hipError_t bin_gather_f64(const FieldPtrs<double>& f, const Geom& g, const BinPtrs& b,
                          const WindowPtrs<double>& win, double* Et, const FluxPlane* fp,
                          hipStream_t st) {
  return launch_gather<double, false>(f, g, b, win, Et, fp, st);
}
hipError_t bin_gather_f32(const FieldPtrs<float>& f, const Geom& g, const BinPtrs& b,
                          const WindowPtrs<float>& win, double* Et, const FluxPlane* fp,
                          hipStream_t st) {
  return launch_gather<float, false>(f, g, b, win, Et, fp, st);
}
// (null 1/eps_r: eps_r = 1 everywhere)
hipError_t gather_epsw_f64(const FieldPtrs<double>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<double>& win, double* out, hipStream_t st) {
  return f.epsinv ? launch_gather<double, true>(f, g, b, win, out, nullptr, st)
                  : launch_gather<double, false>(f, g, b, win, out, nullptr, st);
}
hipError_t gather_epsw_f32(const FieldPtrs<float>& f, const Geom& g, const BinPtrs& b,
                           const WindowPtrs<float>& win, double* out, hipStream_t st) {
  return f.epsinv ? launch_gather<float, true>(f, g, b, win, out, nullptr, st)
                  : launch_gather<float, false>(f, g, b, win, out, nullptr, st);
}
hipError_t gather_batch_f64(const GatherJob<double>* jobs, const int2* order, int nblocks,
                            int reach, bool wide, hipStream_t st) {
  return launch_gather_batch<double>(jobs, order, nblocks, reach, wide, st);
}
hipError_t gather_batch_f32(const GatherJob<float>* jobs, const int2* order, int nblocks,
                            int reach, bool wide, hipStream_t st) {
  return launch_gather_batch<float>(jobs, order, nblocks, reach, wide, st);
}

}  // namespace mlk
