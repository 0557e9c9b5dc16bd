// Entry points of the emulated sweeps: each takes host arrays, lays out what a
// level holds (guarded, so that an access past an end faults), packs the sweep
// data with the library's own kernels and runs a sequence of sweeps.  They
// return 0, or what was found wrong: 1 an access outside the arrays, 2 a watchdog,
// 4 counters or buffer word not ready for the next launch, 8 an entry of the next
// sweep's strip buffer without its sentinel.
#include <algorithm>
#include <type_traits>

#include SMG_SOURCE

using namespace smg;

namespace {

template <class T>
struct Arr {
  T* p;
  size_t n;
  explicit Arr(size_t n_, int fill = 0xff) : n(n_) {
    p = (T*)emu::guarded(n * sizeof(T), fill);
    emu::arrays.push_back({(char*)p, (char*)p + (n * sizeof(T) + 15) / 16 * 16});
  }
  Arr(const double* src, size_t n_) : Arr(n_) {
    for (size_t i = 0; i < n; ++i) p[i] = (T)src[i];
  }
  ~Arr() {
    for (size_t i = 0; i < emu::arrays.size(); ++i)
      if (emu::arrays[i].lo == (char*)p) emu::arrays.erase(emu::arrays.begin() + i--);
    emu::unguard((char*)p, n * sizeof(T));
  }
  Arr(const Arr&) = delete;
};

template <class V>
void sentinels(V* p, size_t n) {
  for (size_t i = 0; i < n; ++i) p[i] = VBits<V>::val(VBits<V>::sent);
}
template <class V>
bool all_sentinels(const V* p, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (VBits<V>::bits(p[i]) != VBits<V>::sent) return false;
  return true;
}
void start(int cap, unsigned long seed) {
  emu::errors = 0;
  emu::cap = (unsigned)cap;
  emu::seed = seed;
}
struct Plain {  // launches without barriers
  Plain() { emu::plain = true; }
  ~Plain() { emu::plain = false; }
};

}  // namespace

#ifdef EMU_WAVEFRONT
namespace {
// A level's scalar sweep data.
template <class E>
struct Level {
  using V = typename WfVal<E>::V;
  Grid g;
  WfTiling t;
  long se;
  Arr<V> h, x, strip;
  Arr<E> pk0, pk1;
  Arr<float> sd;
  Arr<unsigned> par;
  Level(const int* n, int pat, int shape, const double* A, const double* rd, const unsigned short* a16,
        const float* sc)
      : g{n[0], n[1], n[2]}, t(tiling(g, pat, shape)), se(wf_strip_elems(t, pat)), h(g.N()), x(g.N()), strip(2 * se),
        pk0(packs(pat)), pk1(packs(pat)), sd(2 * t.nsk), par(1, 0) {
    Plain plain;
    sentinels(strip.p, 2 * se);
    const long N = g.N();
    if constexpr (sizeof(E) == 2) {
      Arr<__half> a((size_t)pat * N);
      memcpy(a.p, a16, 2 * (size_t)pat * N);
      std::vector<float> r(rd, rd + N);
      launch_wf_pack_h(pat, g, t, 1, a.p, sc, r.data(), pk0.p, sd.p, nullptr);
      launch_wf_pack_h(pat, g, t, -1, a.p, sc, r.data(), pk1.p, sd.p, nullptr);
    } else {
      launch_wf_pack<E>(pat, g, t, 1, A, rd, A, pk0.p, nullptr);
      launch_wf_pack<E>(pat, g, t, -1, A, rd, A, pk1.p, nullptr);
    }
  }
  static WfTiling tiling(const Grid& g, int pat, int shape) {
    WfTiling t;
    wf_tiling(g, pat, &t, shape);
    return t;
  }
  size_t packs(int pat) const { return (size_t)wf_pack_count(pat, sizeof(E)) * t.nsk * 16 / sizeof(E); }
  WfArgs<V> args(int dir) {
    WfArgs<V> a{};
    a.g = g;
    a.t = t;
    a.pk = dir > 0 ? (void*)pk0.p : (void*)pk1.p;
    a.sd = sd.p;
    a.h = h.p;
    a.x = x.p;
    a.strip = strip.p;
    a.par = par.p;
    return a;
  }
  int ready(unsigned word) const {  // after `word` sweeps
    return (par.p[0] != (word & 1u) ? 4 : 0) | (all_sentinels(strip.p + (par.p[0] & 1u ? se : 0), se) ? 0 : 8);
  }
};

template <class E>
int scalar(const int* n, int pat, int shape, int unitd, int ns, const int* dirs, int cap, unsigned long seed,
           const double* A, const double* rd, const unsigned short* a16, const float* sc, const double* h, double* x) {
  using V = typename WfVal<E>::V;
  Level<E> L(n, pat, shape, A, rd, a16, sc);
  Arr<unsigned> ctr(64, 0), err(1, 0);
  int bad = 0;
  for (int k = 0; k < ns; ++k) {
    start(cap, seed + k);
    const long N = L.g.N();
    for (long i = 0; i < N; ++i) {
      L.h.p[i] = (V)h[k * N + i];
      L.x.p[i] = (V)NAN;
    }
    WfArgs<V> a = L.args(dirs[k]);
    a.ctr = ctr.p;
    a.err = err.p;
    if (launch_wavefront<E>(pat, dirs[k], unitd != 0, false, a, nullptr) != hipSuccess) return 64;
    bad |= (emu::errors ? 1 : 0) | (err.p[0] ? 2 : 0) | (ctr.p[0] ? 4 : 0) | L.ready(k + 1);
    for (long i = 0; i < N; ++i) x[k * N + i] = (double)L.x.p[i];
  }
  return bad;
}
}  // namespace

extern "C" int emu_scalar(const int* n, int pat, int shape, int unitd, int ns, const int* dirs, int cap,
                          unsigned long seed, const double* A, const double* rd, const unsigned short* a16,
                          const float* sc, const double* h, double* x) {
  return scalar<EMU_TYPE>(n, pat, shape, unitd, ns, dirs, cap, seed, A, rd, a16, sc, h, x);
}

#ifdef EMU_GROUP
// Several FP64 grids in one launch (arrays one after another); live marks the
// systems that take part.
extern "C" int emu_group(int nsys, const int* dims, int pat, int dir, int order, const int* live, int cap,
                         unsigned long seed, const double* A, const double* rd, const double* h, double* x) {
  std::vector<Level<double>*> L;
  std::vector<WfArgs<double>> segs;
  std::vector<unsigned> tmap;
  long at = 0;
  int most = 0;
  for (int s = 0; s < nsys; ++s) {
    L.push_back(new Level<double>(dims + 3 * s, pat, 0, A + at * pat, rd + at, nullptr, nullptr));
    memcpy(L[s]->h.p, h + at, sizeof(double) * L[s]->g.N());
    at += L[s]->g.N();
    segs.push_back(L[s]->args(dir));
    segs[s].sys = s;
    most = std::max(most, L[s]->t.ntx * L[s]->t.nty);
  }
  auto tiles = [&](int s) { return L[s]->t.ntx * L[s]->t.nty; };
  if (order == 0)
    for (int s = 0; s < nsys; ++s)
      for (int r = 0; r < tiles(s); ++r) tmap.push_back((unsigned)s << 20 | (unsigned)r);
  else
    for (int r = 0; r < most; ++r)
      for (int s = 0; s < nsys; ++s)
        if (r < tiles(s)) tmap.push_back((unsigned)s << 20 | (unsigned)r);
  Arr<unsigned> ctr(64, 0), err(1, 0);
  start(cap, seed);
  if (launch_wavefront_group<double>(pat, dir, segs.data(), nsys, tmap.data(), (unsigned)tmap.size(), 0, live, ctr.p, err.p,
                                     nullptr) != hipSuccess)
    return 64;
  int bad = (emu::errors ? 1 : 0) | (err.p[0] ? 2 : 0) | (ctr.p[0] ? 4 : 0);
  at = 0;
  for (int s = 0; s < nsys; ++s) {
    bad |= L[s]->ready(live[s] ? 1 : 0);
    memcpy(x + at, L[s]->x.p, sizeof(double) * L[s]->g.N());
    at += L[s]->g.N();
    delete L[s];
  }
  return bad;
}

// tile order of a grid of tiles
extern "C" void emu_tile_order(int sh, int ntx, int nty, unsigned* out) {
  for (unsigned k = 0; k < (unsigned)(ntx * nty); ++k) out[k] = sweep_tile(k, sh, ntx, nty);
}
#endif
#endif

#ifdef EMU_BLOCK
namespace {
template <class E>
int block(const int* n, int ns, const int* dirs, int cap, unsigned long seed, const double* A, const double* D,
          const unsigned short* a16, const float* sc, const double* h, double* x) {
  using V = typename WfVal<E>::V;
  const Grid g{n[0], n[1], n[2]};
  WfTiling t;
  bwf_tiling(g, &t);
  const long N = g.N(), se = bwf_strip_elems(t);
  const size_t np = (size_t)bwf_pack_count(sizeof(E)) * t.nsk * 16;
  Arr<char> pk0(np), pk1(np);
  Arr<V> hb(3 * N), xb(3 * N), strip(2 * se);
  Arr<unsigned> ctr(64, 0), err(1, 0), par(1, 0);
  sentinels(strip.p, 2 * se);
  {
    Plain plain;
    for (int d = 0; d < 2; ++d) {
      void* const o = d ? pk1.p : pk0.p;
      if constexpr (sizeof(E) == 2) {
        std::vector<float> r(D, D + 9 * N);
        launch_bwf_pack_h(g, t, d ? -1 : 1, (const __half*)a16, sc, r.data(), o, nullptr);
      } else {
        launch_bwf_pack<E>(g, t, d ? -1 : 1, A, D, (E*)o, nullptr);
      }
    }
  }
  int bad = 0;
  for (int k = 0; k < ns; ++k) {
    start(cap, seed + k);
    for (long i = 0; i < 3 * N; ++i) {
      hb.p[i] = (V)h[3 * N * k + i];
      xb.p[i] = (V)NAN;
    }
    WfArgs<V> a{};
    a.g = g;
    a.t = t;
    a.pk = dirs[k] > 0 ? pk0.p : pk1.p;
    a.h = hb.p;
    a.x = xb.p;
    a.strip = strip.p;
    a.par = par.p;
    a.ctr = ctr.p;
    a.err = err.p;
    if (launch_bwavefront<E>(dirs[k], a, nullptr) != hipSuccess) return 64;
    bad |= (emu::errors ? 1 : 0) | (err.p[0] ? 2 : 0) | (ctr.p[0] || par.p[0] != ((k + 1) & 1u) ? 4 : 0) |
           (all_sentinels(strip.p + (par.p[0] & 1u ? se : 0), se) ? 0 : 8);
    for (long i = 0; i < 3 * N; ++i) x[3 * N * k + i] = (double)xb.p[i];
  }
  return bad;
}
}  // namespace

extern "C" int emu_block(int prec, const int* n, int ns, const int* dirs, int cap, unsigned long seed, const double* A,
                         const double* D, const unsigned short* a16, const float* sc, const double* h, double* x) {
  if (prec == 8) return block<double>(n, ns, dirs, cap, seed, A, D, a16, sc, h, x);
  if (prec == 4) return block<float>(n, ns, dirs, cap, seed, A, D, a16, sc, h, x);
  return block<__half>(n, ns, dirs, cap, seed, A, D, a16, sc, h, x);
}
#endif

#ifdef EMU_LINE
namespace {
// forward from zero into u_a, then backward from u_a into u_b, whose sentinels
// the first sweep wrote, and u_a's again
template <class V>
int line(const int* n, int pat, int cap, unsigned long seed, const double* A, const double* tr, const double* tc,
         const double* f, double* x) {
  const Grid g{n[0], n[1], n[2]};
  const long N = g.N();
  Arr<V> a(A, (size_t)pat * N), r(tr, N), c(tc, N), fv(f, N), ua(N), ub(N);
  sentinels(ua.p, N);
  std::vector<int> tiles;
  LgsArgs<V> l{};
  l.ntile = lgs_plan(g, pat, sizeof(V), &l.K, &tiles);
  if (l.ntile != (int)tiles.size() || l.ntile > lgs_reserve(g, pat)) return 32;
  Arr<unsigned> ctr(64, 0), err(1, 0);
  l.g = g;
  l.A = a.p;
  l.rden = r.p;
  l.cp = c.p;
  l.f = fv.p;
  l.tmap = tiles.data();
  l.ctr = ctr.p;
  l.err = err.p;
  int bad = 0;
  for (int k = 0; k < 2; ++k) {
    start(cap, seed + k);
    l.uold = k ? ua.p : nullptr;
    l.x = k ? ub.p : ua.p;
    l.next = k ? ua.p : ub.p;
    if (launch_lgs<V>(pat, k ? -1 : 1, k == 0, l, nullptr) != hipSuccess) return 64;
    bad |= (emu::errors ? 1 : 0) | (err.p[0] ? 2 : 0) | (ctr.p[0] || ctr.p[1] ? 4 : 0) |
           (all_sentinels(l.next, N) ? 0 : 8);
    for (long i = 0; i < N; ++i) x[k * N + i] = (double)l.x[i];
  }
  return bad;
}
}  // namespace

extern "C" int emu_line(int prec, const int* n, int pat, int cap, unsigned long seed, const double* A, const double* tr,
                        const double* tc, const double* f, double* x) {
  return prec == 8 ? line<double>(n, pat, cap, seed, A, tr, tc, f, x) : line<float>(n, pat, cap, seed, A, tr, tc, f, x);
}
#endif
