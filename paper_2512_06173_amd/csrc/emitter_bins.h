// The bins of the gather and the scatter, formed on the host when emitters are added.  Plain
// C++ without the GPU; every list is sized before it is filled, so that the set-up takes a
// fixed number of allocations however many emitters there are.  The whole set-up of 100,000
// emitters in 256^3 cells takes 22 ms (FP64 17.5), of a million 290; 56 (57) and 700 (810) with
// a list of pairs per emitter and the records put in order on the host.
#pragma once
#include <algorithm>
#include <cmath>
#include <climits>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace mlk {

// A scatter pair: emitter e (its place in the gather's order where the amplitudes are put in
// that order, see scatter_amps), where its record's weights lie (in 16-byte units from the first
// record), and per axis the offset of its union window in the bin, o = (window offset) -
// (bin-local cell), as a signed byte at bit 8 a of off.
struct PairDesc {
  int e;
  int off;
  unsigned rec;
  int pad;
};
static_assert(sizeof(PairDesc) == 16, "a pair is loaded as one int4");

// What a wavefront of the scatter takes: a bin and its pairs [first, end) (equal: nothing);
// shared: the wavefronts of the workgroup take the same bin together.
struct BinSlot {
  int bin, first, end, shared;
};
static_assert(sizeof(BinSlot) == 16, "a slot is loaded as one int4");

struct BinSpec {
  int n[3], periodic[3];  // grid
  int G[3], S[3];         // cells of a gather and of a scatter bin
  int halo;               // most that a window may reach beyond its centre cell
  int light_max;          // gather bins of at most this many emitters are light
  int waves, limit;       // wavefronts of a scatter workgroup; pairs beyond which they share a bin
  bool deal;              // deal the emitters of a gather bin to wavefronts by LDS bank (FP32)
  bool places;            // pairs name an emitter by its place
  unsigned rec16, w16;    // 16-byte units of a record, and those before its weights
};

struct EmitterBins {
  int nb[3] = {};                             // scatter bins per axis
  int gdense = 0, glight0 = 0, reach = 0;     // see BinPtrs
  std::vector<int> gorg, gstart, gem;         // gather bins: origin (3 each), CSR, emitters
  std::vector<float> gwork, swork;            // work of a gather / scatter workgroup
  std::vector<unsigned char> wplane[3];       // planes that some window reaches
  std::vector<BinSlot> sbin;                  // spec.waves to a workgroup
  std::vector<PairDesc> spair;
};

// pos: 3 per emitter; org, len: first point and points of its union window per axis.
// Returns null, or what the emitters do not fit.
inline const char* build_emitter_bins(const BinSpec& sp, int M, const double* pos, const int* org,
                                      const int* len, EmitterBins& out) {
  const int* n = sp.n;
  auto wrap = [&](int q, int a) {
    q %= n[a];
    return q < 0 ? q + n[a] : q;
  };
  // gather: emitters by the bin of their (unwrapped) centre cell, z slowest
  struct Bin3 {
    int b[3];
  };
  std::vector<Bin3> gb(M);
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
  out.reach = 0;
  for (int a = 0; a < 3; ++a) out.wplane[a].assign(n[a], 0);
  for (int e = 0; e < M; ++e)
    for (int a = 0; a < 3; ++a) {
      const int c = (int)std::floor(pos[3 * (size_t)e + a]), o = org[3 * (size_t)e + a],
                L = len[3 * (size_t)e + a];
      const int b = (c >= 0 ? c : c - sp.G[a] + 1) / sp.G[a];
      gb[e].b[a] = b;
      lo[a] = std::min(lo[a], b);
      hi[a] = std::max(hi[a], b);
      out.reach = std::max(out.reach, std::max(c - o, o + L - 1 - c));
      for (int d = 0, q = sp.periodic[a] ? wrap(o, a) : o; d < L; ++d, ++q) {
        if (sp.periodic[a] && q == n[a]) q = 0;
        if (q >= 0 && q < n[a]) out.wplane[a][q] = 1;
      }
    }
  if (out.reach > sp.halo) return "a kernel window reaches too many cells";
  std::vector<int> order(M);
  double boxes = 1.0;
  for (int a = 0; a < 3; ++a) boxes *= M ? (double)hi[a] - lo[a] + 1.0 : 0.0;
  if (boxes <= 4.0 * M + 65536.0) {  // a counting sort over the bins between lo and hi
    const int w0 = M ? hi[0] - lo[0] + 1 : 0, w1 = M ? hi[1] - lo[1] + 1 : 0;
    auto key = [&](int e) {
      const int* b = gb[e].b;
      return (size_t)(b[0] - lo[0]) + (size_t)w0 * ((b[1] - lo[1]) + (size_t)w1 * (b[2] - lo[2]));
    };
    std::vector<int> at((size_t)boxes + 1, 0);
    for (int e = 0; e < M; ++e) ++at[key(e) + 1];
    for (size_t q = 1; q < at.size(); ++q) at[q] += at[q - 1];
    for (int e = 0; e < M; ++e) order[at[key(e)]++] = e;
  } else {
    for (int e = 0; e < M; ++e) order[e] = e;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
      const int *p = gb[x].b, *q = gb[y].b;
      return p[2] != q[2] ? p[2] < q[2] : (p[1] != q[1] ? p[1] < q[1] : p[0] < q[0]);
    });
  }
  auto same = [&](int x, int y) {
    return gb[x].b[0] == gb[y].b[0] && gb[x].b[1] == gb[y].b[1] && gb[x].b[2] == gb[y].b[2];
  };
  std::vector<int> cut;
  cut.reserve((size_t)M + 1);
  for (int q = 0; q < M; ++q)
    if (q == 0 || !same(order[q], order[q - 1])) cut.push_back(q);
  cut.push_back(M);
  // light bins after the others, keeping the order within each kind: the heavier bins are
  // dispatched first
  const int nbin = (int)cut.size() - 1;
  out.gorg.resize((size_t)3 * nbin);
  out.gstart.resize(nbin + 1);
  out.gem.resize(M);
  int bin = 0, em = 0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int b = 0; b < nbin; ++b) {
      if ((cut[b + 1] - cut[b] <= sp.light_max) != (pass == 1)) continue;
      for (int a = 0; a < 3; ++a)
        out.gorg[(size_t)3 * bin + a] = gb[order[cut[b]]].b[a] * sp.G[a];
      out.gstart[bin++] = em;
      for (int q = cut[b]; q < cut[b + 1]; ++q) out.gem[em++] = order[q];
    }
    if (pass == 0) out.gdense = bin;
  }
  out.gstart[nbin] = M;
  // the light bins' emitters are one run of gem (the gather serves them without a tile)
  out.glight0 = out.gstart[out.gdense];
  // work of workgroup q of the tiled bins (taken through the kernel's XCD order): its
  // emitter count
  const int nd = out.gdense, q8 = nd / 8;
  out.gwork.assign(nd, 0.f);
  for (int q = 0; q < nd; ++q) {
    const int b = q < 8 * q8 ? (q % 8) * q8 + q / 8 : q;
    out.gwork[q] = (float)(out.gstart[b + 1] - out.gstart[b]);
  }
  // FP32 gather: the eight emitters of a wavefront read their window rows from the
  // staged tile at the same row and plane offsets, so lane i of emitter m reads word
  // s_m + i + (a common offset), and emitters whose windows start in the same LDS
  // banks conflict.  The bank of s_m is its tile index mod 64.  Within a staged bin, the
  // emitters are sorted by that bank and dealt to the wavefronts with a stride, so
  // those of one wavefront (and of each half) start in banks spread around the 64.
  // Only the assignment of emitters to lanes changes, not any result.
  if (sp.deal) {
    const int R = out.reach <= 3 ? 3 : 4, tx = sp.G[0] + 2 * sp.halo, ps = tx * (sp.G[1] + 2 * R);
    std::vector<int> dealt(M);
    for (int b = 0; b < nd; ++b) {
      const int q0 = out.gstart[b], q1 = out.gstart[b + 1], m = q1 - q0;
      const int* g0 = &out.gorg[(size_t)3 * b];
      const int x0 = g0[0] - sp.halo, y0 = g0[1] - R, z0 = g0[2] - R;
      auto bank = [&](int e) {
        const int* o = org + 3 * (size_t)e;
        return ((o[0] - x0) + tx * (o[1] - y0) + ps * (o[2] - z0)) & 63;
      };
      int at[65] = {};
      for (int q = q0; q < q1; ++q) ++at[bank(out.gem[q]) + 1];
      for (int k = 1; k <= 64; ++k) at[k] += at[k - 1];
      for (int q = q0; q < q1; ++q) dealt[at[bank(out.gem[q])]++] = out.gem[q];
      const int nw = (m + 7) / 8;
      int q = q0;
      for (int w = 0; w < nw; ++w)
        for (int k = 0; k < 8; ++k)
          if (w + k * nw < m) out.gem[q++] = dealt[w + k * nw];
    }
  }

  // scatter: the union window of each emitter split, per axis, into runs inside one bin:
  // consecutive window offsets on consecutive cells.  A pair is one run per axis; a window
  // wraps inside a bin only on a periodic axis no longer than the bin, where it gives
  // several runs.
  struct Run {
    int bin, o;  // window offset - bin-local cell
  };
  constexpr int kRuns = 16;  // a window has at most eight points
  for (int a = 0; a < 3; ++a) out.nb[a] = (n[a] + sp.S[a] - 1) / sp.S[a];
  auto runs_of = [&](int e, int a, Run* r) {
    const int L = std::min(len[3 * (size_t)e + a], kRuns);
    int k = 0;
    for (int d = 0, w = wrap(org[3 * (size_t)e + a], a); d < L;) {
      const int b = w / sp.S[a], l = w - b * sp.S[a];
      const int c = std::min(L - d, std::min(sp.S[a] - l, n[a] - w));
      r[k++] = {b, d - l};
      d += c;
      w = w + c == n[a] ? 0 : w + c;
    }
    return k;
  };
  auto each_pair = [&](int e, auto&& f) {
    Run x[kRuns], y[kRuns], z[kRuns];
    const int nx = runs_of(e, 0, x), ny = runs_of(e, 1, y), nz = runs_of(e, 2, z);
    for (int k = 0; k < nz; ++k)
      for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i)
          f((size_t)x[i].bin + (size_t)out.nb[0] * (y[j].bin + (size_t)out.nb[1] * z[k].bin),
            (x[i].o & 255) | (y[j].o & 255) << 8 | (z[k].o & 255) << 16);
  };
  const size_t nball = (size_t)out.nb[0] * out.nb[1] * out.nb[2];
  std::vector<size_t> at(nball + 1, 0);
  for (int e = 0; e < M; ++e) each_pair(e, [&](size_t b, int) { ++at[b + 1]; });
  size_t nslot = 0;
  for (size_t b = 1; b <= nball; ++b) {
    nslot += at[b] > 0;
    at[b] += at[b - 1];
  }
  if (at[nball] > (size_t)INT32_MAX) return "too many emitter-bin pairs";
  if ((size_t)M * sp.rec16 > UINT32_MAX) return "too many emitters";
  std::vector<BinSlot> slots;
  slots.reserve(nslot);
  for (size_t b = 0; b < nball; ++b)
    if (at[b + 1] > at[b]) slots.push_back({(int)b, (int)at[b], (int)at[b + 1], 0});
  // emitters in gather order, so that neighbouring pairs touch neighbouring windows
  out.spair.resize(at[nball]);
  for (int q = 0; q < M; ++q) {
    const int e = out.gem[q];
    each_pair(e, [&](size_t b, int off) {
      out.spair[at[b]++] = {sp.places ? q : e, off, (unsigned)q * sp.rec16 + sp.w16, 0};
    });
  }

  // The launch's order of bins, sp.waves to a workgroup, or a workgroup to a bin of more than
  // sp.limit pairs.  Workgroups go to the eight XCDs in turn, and neighbouring bins share
  // records and lines of E, so each XCD takes an eighth of the bins of both kinds,
  // neighbours in space; within it the heaviest first (in steps of 32 pairs, so that
  // neighbours stay together), as the light ones then fill in behind them.  Work of a bin: its
  // pairs and, in the same unit, what every bin costs.  Where the eighths differ by more
  // than a quarter in work, the heaviest of all go first instead, dealt to the eight in turn.
  const int W = sp.waves, ns = (int)nslot;
  auto work = [&](const BinSlot& b) { return b.end > b.first ? 16 + b.end - b.first : 0; };
  auto heavier = [&](const BinSlot& x, const BinSlot& y) { return work(x) / 32 > work(y) / 32; };
  const int nsh = (int)std::count_if(slots.begin(), slots.end(),
                                     [&](const BinSlot& b) { return b.end - b.first > sp.limit; });
  const int nblk = nsh + (ns - nsh + W - 1) / W;
  // shared bins first, then the others, filled up to whole workgroups
  std::vector<BinSlot> kind;
  kind.reserve((size_t)nsh + (size_t)W * (nblk - nsh));
  for (int pass = 1; pass >= 0; --pass)
    for (BinSlot b : slots) {
      b.shared = b.end - b.first > sp.limit;
      if (b.shared == pass) kind.push_back(b);
    }
  kind.resize((size_t)nsh + (size_t)W * (nblk - nsh), BinSlot{0, 0, 0, 0});
  BinSlot *sh[9], *lt[9];  // where the eighths begin
  double most = 0.0, total = 0.0;
  sh[0] = kind.data();
  lt[0] = kind.data() + nsh;
  for (int x = 0; x < 8; ++x) {
    const int blocks = nblk / 8 + (x < nblk % 8), mine = nsh / 8 + (x < nsh % 8);
    sh[x + 1] = sh[x] + mine;
    lt[x + 1] = lt[x] + (ptrdiff_t)W * (blocks - mine);
    double w = 0.0;
    for (BinSlot* b = sh[x]; b < sh[x + 1]; ++b) w += work(*b);
    for (BinSlot* b = lt[x]; b < lt[x + 1]; ++b) w += work(*b);
    most = std::max(most, w);
    total += w;
  }
  const bool even = most <= 1.25 * total / 8;
  if (even) {
    for (int x = 0; x < 8; ++x) {
      std::stable_sort(sh[x], sh[x + 1], heavier);
      std::stable_sort(lt[x], lt[x + 1], heavier);
    }
  } else {
    std::stable_sort(sh[0], sh[8], heavier);
    std::stable_sort(lt[0], lt[8], heavier);
  }
  out.sbin.resize((size_t)W * nblk);
  out.swork.resize(nblk);
  for (int b = 0; b < nblk; ++b) {
    const BinSlot* p;
    int step = 1;  // of a workgroup's wavefronts
    if (even) {
      const int x = b % 8, q = b / 8, mine = (int)(sh[x + 1] - sh[x]);
      p = q < mine ? sh[x] + q : lt[x] + (ptrdiff_t)W * (q - mine);
      step = q >= mine;
    } else {
      p = b < nsh ? sh[0] + b : lt[0] + (ptrdiff_t)W * (b - nsh);
      step = b >= nsh;
    }
    int w = 0;
    for (int k = 0; k < W; ++k) {
      out.sbin[(size_t)W * b + k] = p[k * step];
      w = std::max(w, work(p[k * step]) / 32);
    }
    out.swork[b] = (float)w;
  }
  return nullptr;
}

}  // namespace mlk
