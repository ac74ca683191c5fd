// Internal definitions shared by the HIP sources of libmlk (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace mlk {

constexpr int kMaxWin = 8;      // kernel window points per axis (R*sigma <= 3.5 cells)
constexpr int kHalo = 4;        // reach of a window beyond its centre cell (R*sigma + 1/2)
constexpr int kMaxSources = 8;  // soft sources per simulation
constexpr int kMaxLevels = 6;   // multilevel emitters: 2..6 levels

// Geometry and boundary description passed by value to every grid kernel.
struct Geom {
  int n[3];          // cells per axis
  int nlo[3];        // CPML thickness on the low face (0 if none)
  int nhi[3];        // CPML thickness on the high face
  int periodic[3];   // 1 if the axis wraps
  int wall[3];       // 1 if the low face is metallic (PEC or CPML-backed)
  int stream;        // 1: new field values are stored past the caches (see stream_stores)
  double dt;
  double inv_dx;
  double dx;
};

// How the sweeps store new field values.  A grid larger than the 256 MB memory-side
// cache stores them nontemporally: they are read again only in the next step, after the
// whole grid has passed (256^3 FP32: 231 -> 224 us a step without emitters, 384^3 756 ->
// 737; 160^3 FP64 160 -> 152).  A grid whose two field sets stay in that cache must not:
// 128^3 FP32 50.6 -> 41.2 us with ordinary stores, 160^3 (197 MB) 79 -> 63, 128^3 FP64
// (201 MB) 86.6 -> 83.9; from 226 MB on nontemporal ones win (168^3 FP32 95 against 97,
// 176^3 102 against 113, 128 x 128 x 144 FP64 97 against 106).  Nor must FP32 grids whose rows
// are no whole number of 32-byte sectors: the sectors at the tile edges would reach
// memory in parts (250 x 256 x 256 without CPML 264 -> 199 us with ordinary stores, 333 x
// 200 x 200 272 -> 241); FP64 rows, twice as long, show no such loss.
inline int stream_stores(const int n[3], size_t esz) {
  const double bytes = 12.0 * n[0] * n[1] * n[2] * (double)esz;
  return bytes > 208e6 && (esz == 8 || (size_t)n[0] * esz % 32 == 0);
}

// Store of a new field value, past the caches (NT) or not.  The sweep kernels exist in
// both forms: one kernel that branches on the grid's flag at every store ran 2% slower
// (256^3 and 384^3).
template <bool NT, typename T>
__device__ __forceinline__ void store_field(T* p, T v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// XCD-aware order: hardware hands consecutive workgroups to the 8 XCDs in turn;
// map them so that each XCD gets a contiguous range of work items (tiles, bins,
// rows), whose neighbours then meet in the same L2.
__device__ __forceinline__ int xcd_block(int bid, int nblocks) {
  const int q8 = nblocks / 8;
  return bid < 8 * q8 ? (bid % 8) * q8 + bid / 8 : bid;
}

// Workgroup barrier that orders LDS only: global loads in flight (prefetches)
// stay in flight across it, unlike __syncthreads(), whose fence also waits for
// every outstanding global memory operation.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__host__ __device__ inline size_t cell_index(const Geom& g, int i, int j, int k) {
  return (size_t)i + (size_t)g.n[0] * ((size_t)j + (size_t)g.n[1] * (size_t)k);
}

// CPML layer membership of index q along axis a (both the integer and the
// half-integer positions of the layers are stored in the same planes).
__host__ __device__ inline bool in_layer(const Geom& g, int a, int q) {
  return q < g.nlo[a] || q >= g.n[a] - g.nhi[a];
}

// Compressed layer index along axis a.
__host__ __device__ inline int layer_index(const Geom& g, int a, int q) {
  return q < g.nlo[a] ? q : q - (g.n[a] - g.nhi[a]) + g.nlo[a];
}

// Index into the psi array of derivative axis a (that axis compressed to its layers).
__host__ __device__ inline size_t psi_index(const Geom& g, int a, int i, int j, int k) {
  int q[3] = {i, j, k};
  int d[3] = {g.n[0], g.n[1], g.n[2]};
  q[a] = layer_index(g, a, q[a]);
  d[a] = g.nlo[a] + g.nhi[a];
  return (size_t)q[0] + (size_t)d[0] * ((size_t)q[1] + (size_t)d[1] * (size_t)q[2]);
}

__host__ __device__ inline size_t psi_size(const Geom& g, int a) {
  size_t s = 1;
  for (int b = 0; b < 3; ++b) s *= (size_t)(b == a ? g.nlo[a] + g.nhi[a] : g.n[b]);
  return s;
}

// Field storage of one precision.  All CPML psi arrays of a field buffer live
// in one allocation (see psi_offset) and all CPML coefficient tables in another
// (see tab_offset), so a kernel needs two pointers for them.
template <typename T>
struct FieldPtrs {
  T* E[3];
  T* H[3];
  const T* epsinv;
  T* psi;
  const T* tab;
};

__host__ __device__ inline bool has_cpml(const Geom& g, int a) { return g.nlo[a] + g.nhi[a] > 0; }

// psi arrays: for each axis a with a CPML, in axis order, four arrays of
// psi_size(g, a) values: E of the lower-numbered other component, E of the
// higher, then H of the lower and of the higher.  field: 0 = E, 1 = H.
__host__ __device__ inline size_t psi_offset(const Geom& g, int field, int c, int a) {
  size_t off = 0;
  for (int b = 0; b < a; ++b)
    if (has_cpml(g, b)) off += 4 * psi_size(g, b);
  const int lower = a == 0 ? 1 : 0;
  return off + (size_t)(2 * field + (c == lower ? 0 : 1)) * psi_size(g, a);
}

__host__ __device__ inline size_t psi_total(const Geom& g) {
  size_t t = 0;
  for (int a = 0; a < 3; ++a)
    if (has_cpml(g, a)) t += 4 * psi_size(g, a);
  return t;
}

// CPML tables: for each axis with a CPML, in axis order, b, c and 1/kappa, each
// at the n integer positions then the n half-integer positions.
__host__ __device__ inline size_t tab_offset(const Geom& g, int a) {
  size_t off = 0;
  for (int b = 0; b < a; ++b)
    if (has_cpml(g, b)) off += 6 * (size_t)g.n[b];
  return off;
}

__host__ __device__ inline size_t tab_total(const Geom& g) {
  size_t t = 0;
  for (int a = 0; a < 3; ++a)
    if (has_cpml(g, a)) t += 6 * (size_t)g.n[a];
  return t;
}

// Half-open box of cells [lo, hi) per axis.
struct Box {
  int lo[3];
  int hi[3];
};

struct Source {
  int kind;  // 0 plane, 1 point
  int axis, index, comp;
  int ijk[3];
  double amp, omega, tau, t0;
};

struct SourceSet {
  int count;
  Source s[kMaxSources];
};

// Kernel windows of the emitters.  For emitter m, axis a and position variant v
// (v = 0: integer positions, v = 1: half-integer positions; component c uses
// v = 1 on its own axis and v = 0 on the others), slot q = m*6 + 2a + v holds
// the first (unwrapped) index lo[q], the length len[q] <= kMaxWin and the
// normalised 1-D weights w[q*kMaxWin ...].
// The same window in the form the binned kernels stage in LDS.  Per axis the
// union of the two position variants starts at org[a] and spans n[a] <= kMaxWin
// points (the integer points of [r - R sigma - 1/2, r + R sigma]); wr[a][d][v] is
// the weight of variant v at point org[a] + d, zero outside that variant's
// window, so loops over the union need no bounds checks.
template <typename T>
struct alignas(16) WinRec {
  int org[3];
  int n[3];
  int pad[2];
  T wr[3][kMaxWin][2];
};

template <typename T>
struct WindowPtrs {
  const int* lo;
  const int* len;
  const T* w;
  const double* gamma;
  const WinRec<T>* rec;  // [M], in the order of gbin_em (see BinPtrs)
};

__host__ __device__ inline int win_slot(int m, int a, int v) { return m * 6 + 2 * a + v; }


struct TlsPtrs {
  int count;
  const int* gid;          // [M] emitter id of each two-level emitter
  const double* omega0;    // [M]
  const double* dip;       // [3M]
  double* rho;             // [3M] rho11, Re rho01, Im rho01
};

// Multilevel emitters on the device, structure-of-arrays over the slots
// (slot = entry index; slots are grouped by level count).  Matrices sit in a
// kMaxLevels x kMaxLevels frame: entry (a, b) of slot m is at
// (a * kMaxLevels + b) * count + m (complex: re at 2q, im at 2q + 1).
struct MlDev {
  int count;
  const int* gid;       // [count] emitter id
  const double* en;     // [kMaxLevels][count] H0 eigenvalues
  const double* M;      // [kMaxLevels^2][count] real symmetric
  const double* dip;    // [3][count]
  const double* gphi;   // [count]
  double* rho;          // [2 kMaxLevels^2][count]
};

// Number of the step that a launch belongs to: the device's counter, which moves on when the
// last step of a call is closed, plus the steps of the call before this one.  Nothing is
// fixed when the launch is made, so a call that was captured replays as the steps that follow.
struct StepNo {
  int64_t* counter;
  int64_t ahead;
  // (a scalar load: no launch that uses the number moves the counter before every wavefront
  // has read it, and as a scalar it costs emitter kernels neither registers nor VALU divisions)
  __device__ __forceinline__ int64_t get() const {
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(4))) int64_t*)counter + ahead;
#else
    return *counter + ahead;
#endif
  }
};

struct Series {
  double* probe;       // [nprobe][cap]
  int nprobe;
  int probe_comp[16];
  int64_t probe_idx[16];
  int64_t cap;
  double* pop;         // [records][npop]
  int pop_every;
  int64_t npop;
  int64_t pop_cap;     // records
  // non-finite watchdog: 0 while every checked value is finite, else 1 + the first
  // step at which an emitter state, dipole rate, probe sample or flux value was not
  unsigned long long* numeric;
};

// The record of the population series that a step fills; null where it records none, and past
// the room that the host has made (only replays of a captured call get there).
__device__ __forceinline__ double* pop_record(const Series& ser, const StepNo& step) {
  if (ser.pop_every <= 0) return nullptr;
  const int64_t n = step.get();
  if (n % ser.pop_every != 0) return nullptr;
  const int64_t r = n / ser.pop_every;
  return r < ser.pop_cap ? ser.pop + r * ser.npop : nullptr;
}

// Record step n as the first non-finite one.  Steps n - 1 and n can be checked by the
// same launch, so the earliest of the competing records is kept.
__device__ __forceinline__ void flag_nonfinite(const Series& ser, int64_t n) {
  if (!ser.numeric) return;
  const unsigned long long v = (unsigned long long)n + 1ull;
  unsigned long long old = 0ull;  // expected: nothing recorded yet
  for (;;) {
    const unsigned long long seen = atomicCAS(ser.numeric, old, v);
    if (seen == old || (seen != 0ull && seen <= v)) return;
    old = seen;  // a later step got in first: replace it
  }
}

struct FluxPlane {
  int on;
  int axis, index;
  double* Eu0;      // saved E_u^n on the plane (FP64)
  double* Ev0;
  double* partial;  // per-block partial sums
  int nblocks;
  double* series;   // [cap]
  double* total;    // running dt * sum F
};

// Travelling pulse of the classical-path mode: amp f(t - (z - z0)) pol.
struct WaveDesc {
  double pol[3];
  double amp, omega, tau, t0, z0;
};

// Field of the classical-path steps of one launch: a pulse, or rows of an array.
struct PrescribedField {
  int wave;
  const double* Et;  // wave = 0: M x 3 per step, emitter-id order
  size_t stride;     // doubles per step
  WaveDesc w;        // wave = 1: the pulse, at t_start + (q0 + q) dt in step q
  double t_start;
  int64_t q0;
  const double* pos;    // [3M]
  const double* gamma;  // [M]
};

// Discrete field energy W^n, recorded every `every` steps (0: off).
struct EnergyRec {
  int every;
  double* partial;  // per-block partial sums (FP64)
  int nblocks;
  double* series;   // [cap]
  int64_t cap;      // records that the series has room for
  double dv;        // cell volume dx^3
};

// One Lorentz or Drude pole over a cell box: P^{n+1} (1 + g) = a P^n - b P^{n-1} + c E^n.
struct PoleDev {
  int lo[3], n[3];    // box origin and extent (cells)
  double a, b, c, g1; // 2 - kappa w0^2 dt^2, 1 - g, sigma w0^2 dt^2, 1 + g (g = gamma dt / 2)
  void* P;            // P^n, 3 x box cells of the field type, component-major, x fastest
  void* Q;            // P^n - P^{n-1}; after the pre-sweep pass P^{n+1} - P^n
};

// Single-mode cavity that replaces the grid: mode state and coupling.
struct CavityDev {
  double* st;       // q_x, q_y, p_x, p_y, d_x, d_y (FP64)
  double* scratch;  // two more mode states (12 doubles) for the steps of one call
  double* partial;  // two sets of npart per-block partial sums of <mu> + (dt/2) mu_dot, x and y
  int npart;
  double w, V, eps; // mode frequency, effective volume, eps = w / sqrt(V)
};

// Cell (index along axis a; iu, iv along the two others in cyclic order) of a plane.
__device__ __forceinline__ size_t plane_cell(const Geom& g, int a, int index, int iu, int iv) {
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  int q[3];
  q[a] = index;
  q[u] = iu;
  q[v] = iv;
  return cell_index(g, q[0], q[1], q[2]);
}

// Saves E_u^n, E_v^n of plane cell t (the flux needs E^n after the sweep).
template <typename T>
__device__ __forceinline__ void flux_save_body(const FieldPtrs<T>& f, const Geom& g,
                                               const FluxPlane& fp, int t) {
  const int a = fp.axis, u = (a + 1) % 3, v = (a + 2) % 3;
  const int nu = g.n[u], nv = g.n[v];
  if (t >= nu * nv) return;
  const int iu = t % nu, iv = t / nu;
  const size_t id = plane_cell(g, a, fp.index, iu, iv);
  fp.Eu0[t] = (double)f.E[u][id];
  fp.Ev0[t] = (double)f.E[v][id];
}

// Partial flux of block b of nb: 256 threads a block, grid-stride over the plane,
// summed in FP64 in red (256 doubles of LDS) in a fixed order, so the partials do not
// depend on the launch that forms them.  Threads from 256 on (a larger block) only
// take part in the barriers.
template <typename T>
__device__ __forceinline__ void flux_partial_sum(const FieldPtrs<T>& f, const Geom& g,
                                                 const FluxPlane& fp, int b, int nb,
                                                 double* red) {
  const int a = fp.axis, u = (a + 1) % 3, v = (a + 2) % 3;
  const int nu = g.n[u], nv = g.n[v];
  const int tid = threadIdx.x;
  if (tid < 256) {
    double s = 0.0;
    for (int t = b * 256 + tid; t < nu * nv; t += nb * 256) {
      const int iu = t % nu, iv = t / nu;
      const size_t id = plane_cell(g, a, fp.index, iu, iv);
      const size_t jd = plane_cell(g, a, fp.index - 1, iu, iv);
      const double Eu = 0.5 * (fp.Eu0[t] + (double)f.E[u][id]);
      const double Ev = 0.5 * (fp.Ev0[t] + (double)f.E[v][id]);
      const double Hv = 0.5 * ((double)f.H[v][id] + (double)f.H[v][jd]);
      const double Hu = 0.5 * ((double)f.H[u][id] + (double)f.H[u][jd]);
      s += Eu * Hv - Ev * Hu;
    }
    red[tid] = s;
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) fp.partial[b] = red[0];
}


// Binned emitter phase.
// Gather bins: every emitter belongs to the bin of its centre cell; the
// workgroup of a bin stages the bin plus the windows' reach.
// Scatter bins: every (bin, emitter) pair whose window touches the bin.
// Gather bins of at most a few emitters ("light" bins) come after the others and
// stage nothing.
struct BinPtrs {
  int nbx, nby, nbz;        // scatter bins per axis
  int ngather;              // gather bins holding at least one centre
  int gdense;               // bins [0, gdense) stage their tile, the rest are light
  int reach;                // cells that a window reaches beyond its centre cell, at most
  int glight0, nlight;      // gbin_em[glight0 .. glight0 + nlight): the light bins' emitters
  const int* gbin_org;      // [3*ngather] bin origin in unwrapped cells (centre-cell frame)
  const int* gbin_start;    // [ngather+1] CSR into gbin_em
  const int* gbin_em;       // emitter ids; the record of gbin_em[q] is rec[q]
  int nscatter;             // workgroups of the scatter, kScWaves bins each
  const int4* sbin;         // [kScWaves*nscatter] bin, first and end pair (equal: no bin),
                            // 1 if the four wavefronts of the workgroup share the bin
  const int4* sbin_pair;    // one PairDesc per (emitter, bin) pair
  int nem;                  // emitters
  double* amp;              // [3 nem] amplitudes in the order of gbin_em, or null (see scatter_amps)
};

// A batch kernel's job, read from its table through the constant address space.
// The tables are written before the launch and only read by kernels, and pointers
// read from constant memory are known to point to global memory, so the kernel
// reaches the fields through global instructions.  Read from an ordinary pointer,
// the job's pointers would be generic: the compiler would emit flat instructions,
// which also count against the LDS and scalar wait counter.  (The host pass only
// parses kernels; it reads the table directly.)
template <typename J>
__device__ __forceinline__ J load_job(const J* jobs, int j) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((__attribute__((address_space(4))) const J*)jobs)[j];
#else
  return jobs[j];
#endif
}

// scatter bins, one per wavefront
constexpr int kScX = 16, kScY = 4, kScZ = 4, kScWaves = 4;

// ---------------------------------------------------------------- batches
// A batched launch covers the jobs of several domains: job j owns blocks
// [start[j], start[j+1]) of the grid; starts are multiples of 8 so that the
// XCD-aware block order of a job is preserved.
__device__ inline int find_job(const int* start, int njobs, int b) {
  int lo = 0, hi = njobs;  // start[lo] <= b < start[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <typename T>
struct FusedJob {
  FieldPtrs<T> a, b;
  Geom g;
  Box box;
  int kz, tx, ty, ntx, nty, nblocks;  // planes per chunk, tile width and rows, tile grid
};

// Up to four boxes of one sim swept by one launch of the full fused kernel (the
// layer frame around an interior box), passed by value.
template <typename T>
struct FrameJobs {
  FusedJob<T> job[4];
  int start[5];
  int njobs;
};

// The cells of the grid outside an interior box, enumerated in memory order:
// the whole planes below and above the box in z, then, plane by plane inside
// it, the whole rows below and above it in y followed by the two x strips of
// each remaining row.
struct ShellMap {
  Box in;
  int nzlo;              // whole planes below the box
  long long nslab;       // cells in the whole planes (both sides)
  int ylo_rows;          // whole rows below the box, per middle plane
  int full_cells;        // cells in the whole rows of one middle plane
  int strip;             // cells in the two x strips of one row
  int per_plane;         // shell cells of one middle plane
  long long total;       // below 2^31 (checked at launch)
  // reciprocals for the index arithmetic (exact after one correction step)
  double inv_plane, inv_per_plane, inv_nx, inv_strip;
};

// n / d for n < 2^31 from a rounded reciprocal of d: the quotient estimate is off
// by at most one, which the remainder test corrects.
__device__ __forceinline__ unsigned div_by(unsigned n, unsigned d, double inv) {
  unsigned q = (unsigned)((double)n * inv);
  const int r = (int)(n - q * d);
  q = q + (r >= (int)d ? 1u : 0u) - (r < 0 ? 1u : 0u);
  return q;
}

template <typename T>
struct ShellJob {
  FieldPtrs<T> in, out;
  Geom g;
  ShellMap m;
  int nblocks;
};

template <typename T>
struct SourceJob {
  FieldPtrs<T> f;
  Geom g;
  SourceSet src;
  int64_t* step;
  int bx;       // blocks per source
  int nblocks;  // bx * src.count
};

template <typename T>
struct GatherJob {
  FieldPtrs<T> f;
  Geom g;
  BinPtrs bins;
  WindowPtrs<T> win;
  double* Et;
  int nblocks;  // tiled bins, then the light bins' emitters a wavefront each
};

struct TlsJob {
  TlsPtrs tls;
  double dt;
  const double* Et;
  double* mudot;
  const int64_t* pop_off;
  Series ser;
  int64_t* step;
  int nblocks;
};

struct MlJob {
  MlDev ml;
  int first, count;  // slots of one level count
  double dt;
  const double* Et;
  double* mudot;
  const int64_t* pop_off;
  Series ser;
  int64_t* step;
  int nblocks;
};

template <typename T>
struct ScatterJob {
  FieldPtrs<T> f;
  Geom g;
  BinPtrs bins;
  WindowPtrs<T> win;
  const double* mudot;
  int nblocks;  // bins.nscatter
};

template <typename T>
struct FluxJob {
  FieldPtrs<T> f;
  Geom g;
  FluxPlane fp;
  Series ser;
  int64_t* step;
  int nblocks;
};

// Adjoint fields of one sweep: adjoints of E and H, the forward's 1/eps and
// CPML tables, and the adjoint of psi double-buffered (read psi[0], write psi[1]).
template <typename T>
struct AdjSweep {
  T* E[3];
  T* H[3];
  const T* epsinv;
  const T* tab;
  T* psi[2];
  // out of place (fused transposed sweep plus shell passes): the updated
  // adjoint fields go here; null: whole-grid update in place
  T* Eo[3];
  T* Ho[3];
  int kz;  // z planes per workgroup of the fused transposed sweep
  int vacuum;  // eps_r = 1 everywhere: the fused transposed sweep reads no 1/eps_r
};

}  // namespace mlk
