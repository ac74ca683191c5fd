"""Host-side set-up of the gather's and the scatter's bins (csrc/emitter_bins.h), on the CPU:
every window cell lies in exactly one pair of its bin, every emitter in one gather bin and every
bin in one slot, and the set-up allocates no more often for more emitters."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdlib>
#include <new>
static long g_news = 0;
void* operator new(std::size_t n) { ++g_news; if (void* p = std::malloc(n ? n : 1)) return p; throw std::bad_alloc(); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
#include "emitter_bins.h"
using namespace mlk;
static EmitterBins B;
extern "C" const char* run(const int* n, const int* per, const int* G, const int* S, int deal, int limit,
                           int M, const double* pos, const int* org, const int* len, long* news) {
  BinSpec sp{};
  for (int a = 0; a < 3; ++a) { sp.n[a] = n[a]; sp.periodic[a] = per[a]; sp.G[a] = G[a]; sp.S[a] = S[a]; }
  sp.halo = 4; sp.light_max = 8; sp.waves = 4; sp.limit = limit; sp.deal = deal; sp.rec16 = 14; sp.w16 = 2;
  B = EmitterBins();
  g_news = 0;
  const char* e = build_emitter_bins(sp, M, pos, org, len, B);
  *news = g_news;
  return e;
}
extern "C" int size(int what) {
  switch (what) {
    case 0: return (int)B.gorg.size(); case 1: return (int)B.gstart.size(); case 2: return (int)B.gem.size();
    case 3: return (int)B.sbin.size(); case 4: return (int)B.spair.size(); case 5: return (int)B.swork.size();
    case 6: return B.gdense; case 7: return B.glight0; case 8: return B.reach; case 9: return (int)B.gwork.size();
  }
  return B.nb[what - 10];
}
extern "C" const void* data(int what) {
  switch (what) {
    case 0: return B.gorg.data(); case 1: return B.gstart.data(); case 2: return B.gem.data();
    case 3: return B.sbin.data(); case 4: return B.spair.data();
  }
  return B.wplane[what - 5].data();
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bins")
    (d / "h.cpp").write_text(SRC)
    so = str(d / "h.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2512_06173_amd", "csrc"), str(d / "h.cpp"),
                           "-o", so])
    L = C.CDLL(so)
    L.run.restype = C.c_char_p
    L.data.restype = C.c_void_p
    return L


def windows(rng, shape, periodic, m, where):
    """Positions, and union windows as the device forms them (R sigma of 0.5 to 3.5 cells)."""
    shape, rs = np.array(shape), rng.uniform(0.5, 3.5, m)
    lo, hi = np.zeros(3), shape.astype(float)
    pos = rng.uniform(lo, hi, (m, 3)) if where is None else rng.uniform(where[0], where[1], (m, 3))
    for a in range(3):
        if not periodic[a]:
            pos[:, a] = np.clip(pos[:, a], rs + 1, shape[a] - rs - 1)
    org, ln = np.empty((m, 3), np.int32), np.empty((m, 3), np.int32)
    for e in range(m):
        for a in range(3):
            if shape[a] == 1 and periodic[a]:
                org[e, a], ln[e, a] = 0, 1
                continue
            r = pos[e, a]
            q = np.arange(int(np.floor(r)) - 6, int(np.floor(r)) + 7)
            k = q[((q - r) ** 2 <= rs[e] ** 2) | ((q + 0.5 - r) ** 2 <= rs[e] ** 2)]
            org[e, a], ln[e, a] = k[0], k[-1] - k[0] + 1
    return pos, org, ln


def run(lib, shape, periodic, G, deal, limit, pos, org, ln):
    i3 = lambda v: (C.c_int * 3)(*[int(x) for x in v])
    news = C.c_long()
    pos, org, ln = (np.ascontiguousarray(x) for x in (pos, org, ln))
    err = lib.run(i3(shape), i3(periodic), i3(G), i3((16, 4, 4)), int(deal), limit, len(pos),
                  pos.ctypes.data_as(C.c_void_p), org.ctypes.data_as(C.c_void_p),
                  ln.ctypes.data_as(C.c_void_p), C.byref(news))

    def arr(what, dtype, cols):
        n = lib.size(what)
        if n == 0:
            return np.zeros((0, cols), dtype)
        buf = (C.c_char * (n * cols * np.dtype(dtype).itemsize)).from_address(lib.data(what))
        return np.frombuffer(buf, dtype).reshape(n, cols).copy()

    out = dict(err=err, news=news.value, gorg=arr(0, np.int32, 1).reshape(-1, 3),
               gstart=arr(1, np.int32, 1).ravel(), gem=arr(2, np.int32, 1).ravel(),
               sbin=arr(3, np.int32, 4), spair=arr(4, np.int32, 4), blocks=lib.size(5),
               gdense=lib.size(6), glight0=lib.size(7), reach=lib.size(8),
               nb=[lib.size(10 + a) for a in range(3)])
    out["wplane"] = [np.frombuffer((C.c_char * shape[a]).from_address(lib.data(5 + a)),
                                   np.uint8).copy() for a in range(3)]
    return out


CASES = [((64, 48, 40), (0, 0, 0), 300, None), ((37, 23, 21), (0, 0, 0), 900, ((15, 10, 9), (18, 12, 11))),
         ((33, 22, 25), (1, 1, 0), 400, None), ((5, 6, 7), (1, 1, 1), 60, None),
         ((3, 2, 1), (1, 1, 1), 20, None), ((36, 12, 1), (1, 1, 1), 500, None),
         ((1, 16, 20), (1, 1, 1), 64, None), ((900, 700, 800), (0, 0, 0), 40, None),
         ((17, 16, 8), (1, 1, 1), 1, None), ((64, 64, 64), (1, 1, 1), 2500, ((0, 0, 20), (64, 64, 32)))]


@pytest.mark.parametrize("limit", [128, 20])
@pytest.mark.parametrize("deal", [0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_bins_cover_the_windows(lib, case, deal, limit):
    shape, periodic, m, where = CASES[case]
    rng = np.random.default_rng(100 * case + deal)
    G = (16, 8, 8) if deal else (8, 8, 8)
    pos, org, ln = windows(rng, shape, periodic, m, where)
    b = run(lib, shape, periodic, G, deal, limit, pos, org, ln)
    assert b["err"] is None
    # gather: every emitter once, in the bin of its centre cell; light bins behind the others
    assert np.array_equal(np.sort(b["gem"]), np.arange(m)) and b["gstart"][-1] == m
    centre = np.floor(pos).astype(int)
    nbin = len(b["gstart"]) - 1
    for k in range(nbin):
        q0, q1 = b["gstart"][k], b["gstart"][k + 1]
        assert q1 > q0 and (q1 - q0 <= 8) == (k >= b["gdense"])
        for e in b["gem"][q0:q1]:
            assert np.array_equal((centre[e] // G) * G, b["gorg"][k])
    assert len(np.unique(b["gorg"], axis=0)) == nbin
    assert b["glight0"] == b["gstart"][b["gdense"]]
    assert b["reach"] == max(np.max(centre - org), np.max(org + ln - 1 - centre))
    for a in range(3):
        want = np.zeros(shape[a], np.uint8)
        for e in range(m):
            want[(org[e, a] + np.arange(ln[e, a])) % shape[a]] = 1
        assert np.array_equal(b["wplane"][a], want)
    # scatter: every bin with pairs once (four times over where a workgroup shares it)
    assert b["blocks"] * 4 == len(b["sbin"])
    seen = {}
    for w in b["sbin"].reshape(-1, 4, 4):
        if w[0, 3]:
            assert np.all(w == w[0]) and w[0, 2] - w[0, 1] > limit
            w = w[:1]
        for id_, first, end, shared in w:
            if first == end:
                continue
            assert id_ not in seen and (end - first > limit) == bool(shared)
            seen[id_] = (first, end)
    ranges = sorted(seen.values())
    assert [r[0] for r in ranges] == [0] + [r[1] for r in ranges[:-1]] and \
        ranges[-1][1] == len(b["spair"])
    # every window point of every emitter, at its cell, in exactly one pair of that cell's bin
    place = np.empty(m, int)
    place[b["gem"]] = np.arange(m)
    cover = {}
    for id_, (first, end) in seen.items():
        bx, by, bz = id_ % b["nb"][0], id_ // b["nb"][0] % b["nb"][1], id_ // (b["nb"][0] * b["nb"][1])
        base = (16 * bx, 4 * by, 4 * bz)
        at = [place[p[0]] for p in b["spair"][first:end]]
        assert at == sorted(at)  # in the gather's order
        for e, off, rec, _ in b["spair"][first:end]:
            assert rec == 14 * place[e] + 2
            for a in range(3):
                o = (off >> 8 * a & 255 ^ 128) - 128
                S = (16, 4, 4)[a]
                # the weights that cells of the bin read; what lies outside is zero weight
                pts = [(base[a] + l, l + o) for l in range(S)
                       if 0 <= l + o < ln[e, a] and base[a] + l < shape[a]]
                cover.setdefault((e, id_), []).append(pts)
    total = np.zeros(m, int)
    for (e, id_), runs in cover.items():
        for k in range(0, len(runs), 3):
            x, y, z = runs[k:k + 3]
            total[e] += len(x) * len(y) * len(z)
            for a, pts in enumerate((x, y, z)):
                assert pts and all((org[e, a] + d) % shape[a] == c for c, d in pts)
    assert np.array_equal(total, ln.prod(axis=1))


def test_setup_allocates_no_more_often_for_more_emitters(lib):
    """(One vector per emitter took 62 ms for 100,000 emitters in 256^3 cells.)"""
    news = []
    for m in (50, 5000):
        rng = np.random.default_rng(m)
        pos, org, ln = windows(rng, (64, 64, 64), (1, 1, 1), m, None)
        news.append(run(lib, (64, 64, 64), (1, 1, 1), (16, 8, 8), 1, 128, pos, org, ln)["news"])
    # (std::stable_sort takes one buffer a call, 16 calls at most)
    assert max(news) <= 60, news


def test_windows_that_reach_too_far_are_refused(lib):
    pos = np.array([[20.5, 20.5, 20.5]])
    org, ln = np.array([[15, 17, 17]], np.int32), np.array([[8, 7, 7]], np.int32)
    assert run(lib, (64, 64, 64), (0, 0, 0), (8, 8, 8), 0, 128, pos, org, ln)["err"]
