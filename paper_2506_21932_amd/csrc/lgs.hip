// Line Gauss-Seidel over z-columns (Sec. 4.4, "For LGS" paragraph): the
// unknowns of one column (x, y) are updated together.  The right-hand side of
// a column is assembled from the neighbouring columns, then the column's
// tridiagonal system (couplings (0,0,-1), centre, (0,0,+1)) is solved by the
// Thomas algorithm.  Columns are visited in lexicographic (x, y) order
// (forward) or in reverse (backward), as in the GS formulas with the column
// blocks as D.
//
// Setup: k_tri_factor forms the Thomas pivots once per hierarchy (FP64, one
// thread per column): p_0 = b_0, p_z = fma(-a_z, cp_{z-1}, b_z),
// rden_z = 1/p_z, cp_z = c_z * rden_z.
//
// Sweep: a column depends only on columns whose (x, y) come earlier
// in the visiting order and are stencil neighbours (the projected 2D pattern:
// 2d5 for 3d7, 2d9 for 3d19 / 3d27).  In the sheared coordinates
// (x, y' = y + sh*x), sh = 0 for 3d7 and 1 otherwise (the neighbour
// (x-1, y+1) must come first), every such neighbour lies at (dx, dy') with
// dx <= 0, dy' <= 0 and dx + dy' <= -1.  The columns are cut into K x K tiles
// in (x, y'); a tile depends only on the tiles (bx-1, by'), (bx-1, by'-1) and
// (bx, by'-1), so tiles listed by diagonal bx + by' (setup-time table, empty
// tiles left out) are in dependence order.  Persistent workgroups take tiles
// by atomic ticket (every tile's producers hold smaller tickets and are
// already running: the grid always makes progress).  k_lgs_tile walks a
// tile's local hyperplanes lx + ly' = k, K columns each; columns longer than
// its LDS arrays take k_lgs, a column per tile (K = 1).  A column of another
// tile is read back device-coherently, after its sentinel has gone.  The
// backward sweep takes the table (and k_lgs_tile the local hyperplanes) in
// reverse.
// For each column (k_lgs_tile: for the columns of a hyperplane together) a
// workgroup
//   A. assembles the right-hand side, one point per thread:
//      t = f_i; the terms of columns not yet visited (values from before the
//      sweep, plain loads); then the terms of columns of this sweep; each
//      group in canonical order with fma.  The Thomas factors are staged in
//      LDS with the sums;
//   B. solves each column in one lane (forward elimination, back
//      substitution), in the oracle's order of operations;
//   C. stores the column device-coherently and, if asked, writes the sentinel
//      into `next` (the buffer the following sweep will fill).  Every reader
//      of `next` at these points is a column this one waited for, so those
//      reads are complete.
// Waits are bounded: after LGS_SPIN_LIMIT polls, bit 0 of err is set and
// every waiting lane gives up.
#include <algorithm>
#include <utility>
#include <vector>

#include "smg_kernels.h"

namespace smg {

namespace {

constexpr int LGS_NT = 256;                 // k_lgs: threads per workgroup
constexpr int LGS_RESERVE_PTS = 256;        // points per hyperplane of the tiles of lgs_reserve
constexpr unsigned LGS_SPIN_LIMIT = 1u << 21;
constexpr int LT_MAX_GRID = 256;            // k_lgs_tile: one workgroup per CU

__host__ __device__ constexpr int lgs_cwx(int pat) { return pat == 7 ? 1 : 2; }

// does the column at (dx, dy) come later than the current one in the
// visiting order of direction DIR?
__host__ __device__ constexpr bool lgs_later(int dir, int dx, int dy) {
  return dir > 0 ? (dx > 0 || (dx == 0 && dy > 0)) : (dx < 0 || (dx == 0 && dy < 0));
}

template <class V>
__device__ inline V cload(const V* p) {
  using U = typename VBits<V>::U;
  return VBits<V>::val(__hip_atomic_load(reinterpret_cast<const U*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

template <class V>
__device__ inline void cstore(V* p, V v) {
  using U = typename VBits<V>::U;
  __hip_atomic_store(reinterpret_cast<U*>(p), VBits<V>::bits(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded wait until *p no longer holds the sentinel.
template <class V>
__device__ inline V await_value(const V* p, V v, unsigned* err) {
  unsigned spins = 0;
  while (VBits<V>::bits(v) == VBits<V>::sent) {
    if (++spins >= LGS_SPIN_LIMIT) {
      atomicOr(err, 1u);
      break;
    }
    if ((spins & 1023u) == 1023u && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u)) break;
    __builtin_amdgcn_s_sleep(2);
    v = cload(p);
  }
  return v;
}

// Loads of the term of slot S (off-column slots only), issued for all slots
// before any wait: in-grid flag, coefficient, and the neighbour's value (from
// before the sweep for a column later in the order, else device-coherently
// from the output).  A neighbour outside the grid loads the row's own
// position instead; its term is not used.
template <int PAT, int DIR, bool ZG, int S, class V>
__device__ __forceinline__ void lgs_load(bool (&in)[PAT], V (&av)[PAT], V (&uv)[PAT], const LgsArgs<V>& a, long N,
                                         long i, int X, int Y, int Z) {
  constexpr int dx = pat_off(PAT, S, 0), dy = pat_off(PAT, S, 1), dz = pat_off(PAT, S, 2);
  if constexpr (!(dx == 0 && dy == 0) && !(ZG && lgs_later(DIR, dx, dy))) {
    in[S] = in_grid(a.g, X + dx, Y + dy, Z + dz);
    const long j = in[S] ? i + dx * ((long)a.g.ny * a.g.nz) + dy * (long)a.g.nz + dz : i;
    av[S] = a.A[(long)S * N + i];
    if constexpr (lgs_later(DIR, dx, dy))
      uv[S] = a.uold[j];
    else
      uv[S] = cload(a.x + j);
  }
}

// Bounded wait for the value of a column of this sweep that is still the
// sentinel.
template <int PAT, int DIR, int S, class V>
__device__ __forceinline__ void lgs_wait(const bool (&in)[PAT], V (&uv)[PAT], const LgsArgs<V>& a, long i) {
  constexpr int dx = pat_off(PAT, S, 0), dy = pat_off(PAT, S, 1), dz = pat_off(PAT, S, 2);
  if constexpr (!(dx == 0 && dy == 0) && !lgs_later(DIR, dx, dy)) {
    if (in[S] && VBits<V>::bits(uv[S]) == VBits<V>::sent)
      uv[S] = await_value(a.x + i + dx * ((long)a.g.ny * a.g.nz) + dy * (long)a.g.nz + dz, uv[S], a.err);
  }
}

// t = fma(-a_s, u_nbr, t) for slot S if it belongs to the group (OLD: columns
// later in the order) and its neighbour is in the grid.
template <int PAT, int DIR, bool OLD, int S, class V>
__device__ __forceinline__ void lgs_acc(V& t, const bool (&in)[PAT], const V (&av)[PAT], const V (&uv)[PAT]) {
  constexpr int dx = pat_off(PAT, S, 0), dy = pat_off(PAT, S, 1);
  if constexpr (!(dx == 0 && dy == 0) && lgs_later(DIR, dx, dy) == OLD) t = in[S] ? fma(-av[S], uv[S], t) : t;
}

// Right-hand side of point i: f_i, then the group of columns not yet visited
// (omitted for the zero initial guess), then the columns of this sweep, each
// in canonical order.
template <int PAT, int DIR, bool ZG, class V, int... S>
__device__ __forceinline__ V lgs_rhs(const LgsArgs<V>& a, long N, long i, int X, int Y, int Z,
                                     std::integer_sequence<int, S...>) {
  bool in[PAT];
  V av[PAT], uv[PAT];
  V t = a.f[i];
  (lgs_load<PAT, DIR, ZG, S, V>(in, av, uv, a, N, i, X, Y, Z), ...);
  if constexpr (!ZG) (lgs_acc<PAT, DIR, true, S, V>(t, in, av, uv), ...);
  (lgs_wait<PAT, DIR, S, V>(in, uv, a, i), ...);
  (lgs_acc<PAT, DIR, false, S, V>(t, in, av, uv), ...);
  return t;
}

__device__ inline unsigned lgs_take_ticket(unsigned* ctr) {
  __shared__ unsigned s_ticket;
  if (threadIdx.x == 0) s_ticket = atomicAdd(&ctr[0], 1u);
  __syncthreads();
  const unsigned t = s_ticket;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(t);
}

// The last workgroup to finish resets the ticket counters for the next launch.
__device__ inline void lgs_retire(unsigned* ctr) {
  if (threadIdx.x == 0) {
    const unsigned o = atomicAdd(&ctr[1], 1u);
    if (o == gridDim.x - 1) {
      __hip_atomic_store(&ctr[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ctr[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Columns of more than LT_MAX_NZ points: one column at a time, bound by the
// chain of right-hand side, solve (one lane) and hand-off.  64 x 64 x 129, 7-point
// FP64 1.59 ms each way, 19-point FP32 2.10 / 2.38, 27-point FP64 2.51 / 2.99 (a
// form for K x K tiles of shorter columns 1.64, 2.32 / 2.57, 2.51 / 3.03).
template <int PAT, int DIR, class V, bool ZG>
__global__ __launch_bounds__(LGS_NT) void k_lgs(LgsArgs<V> a) {
  constexpr int SH = lgs_cwx(PAT) - 1;
  constexpr int SLO = pat_slot(PAT, 0, 0, -1);
  extern __shared__ __align__(16) unsigned char lgs_smem[];
  const Grid g = a.g;
  const long N = g.N();
  const int nz = g.nz;
  V* ld = reinterpret_cast<V*>(lgs_smem);  // right-hand side, then d', then x
  V* la = ld + nz;                          // coupling to z-1
  V* lr = la + nz;                          // 1 / pivot
  V* lc = lr + nz;                          // c / pivot
  for (;;) {
    const unsigned ticket = lgs_take_ticket(a.ctr);
    if (ticket >= (unsigned)a.ntile) break;
    const int e = a.tmap[DIR > 0 ? (int)ticket : a.ntile - 1 - (int)ticket];
    int X = e >> 16, Y = (e & 0xffff) - SH * X;
    // kept in vector registers, and b below: a scalar form holds every
    // neighbour's test in spilled scalar registers (27 points, backward: 2% of
    // the sweep) and forms the LDS addresses of the solve one by one (10%)
    asm("" : "+v"(X), "+v"(Y));
    const long i0 = ((long)X * g.ny + Y) * nz;
    // A. right-hand sides and staged factors
    for (int Z = threadIdx.x; Z < nz; Z += LGS_NT) {
      const long i = i0 + Z;
      la[Z] = Z > 0 ? a.A[(long)SLO * N + i] : V(0);
      lr[Z] = a.rden[i];
      lc[Z] = a.cp[i];
      ld[Z] = lgs_rhs<PAT, DIR, ZG, V>(a, N, i, X, Y, Z, std::make_integer_sequence<int, PAT>{});
    }
    __syncthreads();
    // B. Thomas solve in one lane, in blocks of 8 points whose LDS reads are
    // issued together.  d'_0 = t_0 * rden_0 comes out of the same formula: the
    // stored coupling to z-1 at z = 0 is +0 and d' starts at +0, so fma(-0, +0,
    // t_0) = t_0 exactly.
    if (threadIdx.x == 0) {
      int b = 0;
      asm("" : "+v"(b));
      V dp = V(0);
      for (int z0 = 0; z0 < nz; z0 += 8) {
        V a8[8], r8[8], d8[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int z = z0 + k < nz ? z0 + k : nz - 1;
          a8[k] = la[b + z];
          r8[k] = lr[b + z];
          d8[k] = ld[b + z];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (z0 + k < nz) {
            dp = fma(-a8[k], dp, d8[k]) * r8[k];
            ld[b + z0 + k] = dp;
          }
        }
      }
      V xv = dp;
      for (int z1 = nz - 2; z1 >= 0; z1 -= 8) {
        V c8[8], d8[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int z = z1 - k >= 0 ? z1 - k : 0;
          c8[k] = lc[b + z];
          d8[k] = ld[b + z];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (z1 - k >= 0) {
            xv = fma(-c8[k], xv, d8[k]);
            ld[b + z1 - k] = xv;
          }
        }
      }
    }
    __syncthreads();
    // C. results out, sentinels for the next sweep
    for (int Z = threadIdx.x; Z < nz; Z += LGS_NT) {
      cstore(a.x + i0 + Z, ld[Z]);
      if (a.next) a.next[i0 + Z] = VBits<V>::val(VBits<V>::sent);
    }
    __syncthreads();  // LDS is refilled by the next column
  }
  lgs_retire(a.ctr);
}

// ---- columns of at most LT_MAX_NZ points -------------------------------------
// The chain of the sweep is one column hyperplane after another (1534 of them
// at 512 x 512), each a right-hand side and a Thomas recurrence of 2 nz
// dependent operations, so everything else is kept out of it.  A workgroup
// holds a tile of K x K columns (K nz points a hyperplane) and steps through
// its 2K - 1 hyperplanes with two barriers each; its waves have roles:
//   point waves, a thread per (lx, z): after the first barrier of a step the
//     terms of this sweep's columns, from LDS, onto a sum of f and the old
//     values that was formed a step earlier; behind the Thomas solve they load
//     the data of the step after next and prepare the next one; they store the
//     columns of the step before, device-coherently, and their sentinels;
//   a Thomas wave, a lane per column: LDS to LDS, the next eight points' reads
//     issued before the current eight are used;
//   a halo wave: the neighbouring tiles' columns the next step needs (one at
//     lx = -1, one each in the rows ly' = -1 and -2), read device-coherently
//     one step ahead and awaited while they hold the sentinel;
// Finished columns stay in an LDS ring of four hyperplanes (the neighbours of
// a column lie one to three hyperplanes back).  The backward sweep mirrors the
// tile.  A hyperplane takes 2.4 us, of which the Thomas solve about half (its
// chain, and LDS reads and writes of 16 bytes).  Forward / backward sweep of a
// 512 x 512 x 64 level, 19-point FP32, before
// (a kernel that did a hyperplane's loads, solves and stores in turn) and with
// this one (MI355X): 10.43 / 11.55 and 3.74 / 3.72 ms; 128 x 128 x 64, 27-point:
// 1.29 / 1.55 and 0.49 / 0.45 ms.  Longer columns gain as much, down to two
// columns a hyperplane: 64 x 64 x 96, 19-point FP64 1.93 / 2.14 and 1.09 / 1.14
// ms, 128^3, 27-point FP64 5.01 / 5.78 and 2.69 / 2.71, FP32 4.41 / 5.27 and
// 1.71 / 1.67 ms; the limit is the halo wave's two values a lane and column.
constexpr int LT_MAX_NZ = 128;
template <class V>
constexpr int lt_pts() {
  return sizeof(V) == 4 ? 512 : 256;  // points per hyperplane (registers per point: two steps' data)
}
__host__ __device__ constexpr int lt_ldp(int nz) { return (nz + 7) / 8 * 8 + 4; }  // column stride of the LDS arrays
__host__ __device__ constexpr int lt_rz(int nz) { return lt_ldp(nz) + 8; }         // ... of the ring (z at z + 4)

// Eight consecutive values (16-byte aligned) of an LDS column.
template <class V>
__device__ __forceinline__ void lt_read8(V (&o)[8], const V* p) {
  typedef V VV __attribute__((ext_vector_type(16 / sizeof(V))));
#pragma unroll
  for (int q = 0; q < 8; q += 16 / (int)sizeof(V)) {
    const VV w = *reinterpret_cast<const VV*>(p + q);
#pragma unroll
    for (int r = 0; r < 16 / (int)sizeof(V); ++r) o[q + r] = w[r];
  }
}
template <class V>
__device__ __forceinline__ void lt_write8(V* p, const V (&o)[8]) {
  typedef V VV __attribute__((ext_vector_type(16 / sizeof(V))));
#pragma unroll
  for (int q = 0; q < 8; q += 16 / (int)sizeof(V)) {
    VV w;
#pragma unroll
    for (int r = 0; r < 16 / (int)sizeof(V); ++r) w[r] = o[q + r];
    *reinterpret_cast<VV*>(p + q) = w;
  }
}

template <int PAT, class V>
struct LtPoint {
  V a[PAT], uo[PAT], t, la, lr, lc;
  bool act, yl, yh;  // is there a point; neighbours at y - 1, y + 1
};

template <int PAT, int DIR, class V, bool ZG>
__global__ __launch_bounds__(lt_pts<V>() + 128) void k_lgs_tile(LgsArgs<V> a) {
  constexpr int SH = lgs_cwx(PAT) - 1, SLO = pat_slot(PAT, 0, 0, -1);
  extern __shared__ __align__(16) unsigned char lgs_smem[];
  using B = VBits<V>;
  const Grid g = a.g;
  const long N = g.N();
  const int nz = g.nz, K = a.K, LDP = lt_ldp(nz), RZ = lt_rz(nz);
  V* const ld = reinterpret_cast<V*>(lgs_smem);  // right-hand side, then d'
  V* const fac = ld + K * LDP;                    // [2][3][K]: coupling to z-1, 1 / pivot, c / pivot
  V* const ring = fac + 6 * K * LDP;              // [4][K + 1]: finished columns, position lx + 1
  const int nsteps = 2 * K - 1;
  const int npw = (K * nz + 63) / 64;  // point waves
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = threadIdx.x % 64;
  // point waves: a thread per (lx, z); the last wave's rest idles
  const bool rest = (int)threadIdx.x >= K * nz;
  const int lx = rest ? K - 1 : (int)threadIdx.x / nz, z = rest ? 0 : (int)threadIdx.x % nz;
  auto ringp = [&](int h, int pos) { return ring + ((h & 3) * (K + 1) + pos) * RZ + 4; };

  for (;;) {
    const unsigned ticket = lgs_take_ticket(a.ctr);
    if (ticket >= (unsigned)a.ntile) break;
    const int e = a.tmap[DIR > 0 ? (int)ticket : a.ntile - 1 - (int)ticket];
    const int bx = e >> 16, by = e & 0xffff;
    // grid column of (lx, ly) in the forward frame; does it exist?
    auto column = [&](int cx, int cy, int& X, int& Y) {
      X = bx * K + (DIR > 0 ? cx : K - 1 - cx);
      Y = by * K + (DIR > 0 ? cy : K - 1 - cy) - SH * X;
      return X >= 0 && X < g.nx && Y >= 0 && Y < g.ny;
    };
    // --- point role (32-bit byte offsets from the plane before the tile's first)
    const int X0 = bx * K > 0 ? bx * K - 1 : 0;
    const long tb = (long)X0 * g.ny * nz;
    const int Xp = bx * K + (DIR > 0 ? lx : K - 1 - lx);
    const int Y0 = by * K + (DIR > 0 ? 0 : K - 1) - SH * Xp;  // y of ly = 0; then DIR steps
    const bool prole = !rest && Xp < g.nx;
    // y of this thread's column at step k; is there one?
    auto at_step = [&](int k, int& Y) {
      const int ly = k - lx;
      Y = Y0 + DIR * ly;
      return prole && (unsigned)ly < (unsigned)K && (unsigned)Y < (unsigned)g.ny;
    };
    const bool xl = Xp > 0, xh = Xp < g.nx - 1, zl = z > 0, zh = z < nz - 1;
    auto inside = [&](const LtPoint<PAT, V>& p, int s) {
      const int dx = pat_off(PAT, s, 0), dy = pat_off(PAT, s, 1), dz = pat_off(PAT, s, 2);
      bool in = p.act;
      if (dx < 0) in = in & xl;
      if (dx > 0) in = in & xh;
      if (dy < 0) in = in & p.yl;
      if (dy > 0) in = in & p.yh;
      if (dz < 0) in = in & zl;
      if (dz > 0) in = in & zh;
      return in;
    };
    // data of step k (every load before the first use; a missing neighbour's
    // value is the point's own and goes unused)
    auto load = [&](LtPoint<PAT, V>& p, int k) {
      int Y;
      p.act = at_step(k, Y);
      p.yl = Y > 0;
      p.yh = Y < g.ny - 1;
      const unsigned o = p.act ? (unsigned)(((Xp - X0) * g.ny + Y) * nz + z) * (unsigned)sizeof(V) : 0u;
      auto at = [&](const V* v, unsigned off) { return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(v + tb) + off); };
#pragma unroll
      for (int s = 0; s < PAT; ++s) {
        const int dx = pat_off(PAT, s, 0), dy = pat_off(PAT, s, 1), dz = pat_off(PAT, s, 2);
        if (dx == 0 && dy == 0) continue;
        const bool later = lgs_later(DIR, dx, dy);
        if (ZG && later) continue;
        p.a[s] = at(a.A + (long)s * N, o);
        if (later)
          p.uo[s] = at(a.uold, inside(p, s) ? o + (unsigned)(((dx * g.ny + dy) * nz + dz) * (int)sizeof(V)) : o);
      }
      p.t = at(a.f, o);
      p.la = at(a.A + (long)SLO * N, o);
      p.lr = at(a.rden, o);
      p.lc = at(a.cp, o);
    };
    // the terms of old values, and the Thomas factors into LDS
    auto stage = [&](LtPoint<PAT, V>& p, int k) {
      if constexpr (!ZG) {
#pragma unroll
        for (int s = 0; s < PAT; ++s) {
          const int dx = pat_off(PAT, s, 0), dy = pat_off(PAT, s, 1);
          if ((dx == 0 && dy == 0) || !lgs_later(DIR, dx, dy)) continue;
          p.t = inside(p, s) ? fma(-p.a[s], p.uo[s], p.t) : p.t;
        }
      }
      if (p.act) {
        V* o = fac + (k & 1) * 3 * K * LDP + lx * LDP + z;
        o[0] = zl ? p.la : V(0);
        o[K * LDP] = p.lr;
        o[2 * K * LDP] = p.lc;
      }
    };
    // the terms of this sweep's columns
    auto rhs = [&](LtPoint<PAT, V>& p, int k) {
      V v[PAT];
#pragma unroll
      for (int s = 0; s < PAT; ++s) {
        const int dx = DIR * pat_off(PAT, s, 0), dy = DIR * pat_off(PAT, s, 1), dz = pat_off(PAT, s, 2);
        if ((dx == 0 && dy == 0) || lgs_later(1, dx, dy)) continue;
        v[s] = ringp(k + dx + dy + SH * dx, lx + 1 + dx)[z + dz];  // forward-frame offset (dx, dy + SH dx)
      }
      V t = p.t;
#pragma unroll
      for (int s = 0; s < PAT; ++s) {
        const int dx = pat_off(PAT, s, 0), dy = pat_off(PAT, s, 1);
        if ((dx == 0 && dy == 0) || lgs_later(DIR, dx, dy)) continue;
        t = inside(p, s) ? fma(-p.a[s], v[s], t) : t;
      }
      if (p.act) ld[lx * LDP + z] = t;
    };
    // --- Thomas role
    const int Xt = bx * K + (DIR > 0 ? lane : K - 1 - lane), Yt = by * K + (DIR > 0 ? 0 : K - 1) - SH * Xt;
    auto solve = [&](int k) {
      const int ly = k - lane;
      if (lane >= K || Xt >= g.nx || (unsigned)ly >= (unsigned)K || (unsigned)(Yt + DIR * ly) >= (unsigned)g.ny) return;
      V* const d = ld + lane * LDP;
      const V* const fa = fac + (k & 1) * 3 * K * LDP + lane * LDP;
      const V *const fr = fa + K * LDP, *const fc = fr + K * LDP;
      V* const out = ringp(k, lane + 1);
      // blocks of 8 points; the next block's reads are issued before this
      // one's chain (behind a last block that is full they bring four values of
      // the LDS column or array after this one, which nothing uses: a clamped
      // address costs 1-2% of the sweep)
      struct Blk {
        V a[8], r[8], d[8];
      };
      const int nb = nz / 8;  // full blocks
      V dp = V(0);
      auto read3 = [&](Blk& b, int z0) {
        lt_read8(b.a, fa + z0);
        lt_read8(b.r, fr + z0);
        lt_read8(b.d, d + z0);
        __builtin_amdgcn_sched_barrier(0);
      };
      // d'_0 = t_0 / pivot_0 comes out of the same formula (coupling and d' are +0)
      auto forward = [&](const Blk& b, int z0, int n) {
        // (a ragged block's last places are written too: they lie past the column)
        V o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const V v = fma(-b.a[q], dp, b.d[q]) * b.r[q];
          dp = q < n ? v : dp;
          o[q] = dp;
        }
        lt_write8(d + z0, o);
        __builtin_amdgcn_sched_barrier(0);
      };
      Blk b0, b1;
      read3(b0, 0);
      int ib = 0;
      for (; ib + 2 <= nb; ib += 2) {
        read3(b1, 8 * ib + 8);
        forward(b0, 8 * ib, 8);
        read3(b0, 8 * ib + 16);
        forward(b1, 8 * ib + 8, 8);
      }
      if (ib < nb) {
        read3(b1, 8 * ib + 8);
        forward(b0, 8 * ib, 8);
        if (nz > 8 * nb) forward(b1, 8 * nb, nz - 8 * nb);
      } else if (nz > 8 * nb) {
        forward(b0, 8 * nb, nz - 8 * nb);
      }
      V xv = dp;  // the last point's value (the ragged block writes it in its place)
      auto read2 = [&](Blk& b, int z0) {
        lt_read8(b.a, fc + z0);
        lt_read8(b.d, d + z0);
        __builtin_amdgcn_sched_barrier(0);
      };
      auto back = [&](const Blk& b, int z0, int n) {
        V o[8];
#pragma unroll
        for (int q = 7; q >= 0; --q) {
          const V v = fma(-b.a[q], xv, b.d[q]);
          xv = q < n ? v : xv;
          o[q] = xv;
        }
        lt_write8(out + z0, o);
        __builtin_amdgcn_sched_barrier(0);
      };
      // points nz - 2 .. 0: the ragged top block, then full blocks
      const int mb = (nz - 1) / 8;
      read2(b0, 8 * mb);
      if (mb > 0) read2(b1, 8 * mb - 8);
      back(b0, 8 * mb, nz - 1 - 8 * mb);
      for (ib = mb - 1; ib >= 1; ib -= 2) {
        read2(b0, 8 * ib - 8);
        back(b1, 8 * ib, 8);
        if (ib >= 2) read2(b1, 8 * ib - 16);
        back(b0, 8 * ib - 8, 8);
      }
      if (ib == 0) back(b1, 0, 8);
    };
    // --- halo role: the neighbouring tiles' columns that step k is the first
    // to need
    constexpr int NC = SH ? 3 : 2;
    V hv[NC][2];
    // column c of step k: (-1, k), (k, -1), (k - 1, -2); k counts along a line
    // of columns, whose first index, step and existing members are kept
    long hbase[NC];
    int hstep[NC];
    unsigned hmask[NC];
    auto halo_plan = [&] {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int cx = c == 0 ? -1 : (c == 1 ? 0 : -1), cy = c == 0 ? 0 : -c;
        int X, Y;
        column(cx, cy, X, Y);
        hbase[c] = ((long)X * g.ny + Y) * nz;
        hstep[c] = DIR * (c == 0 ? 1 : g.ny - SH) * nz;
        hmask[c] = 0;
        for (int k = 0; k < K; ++k) hmask[c] |= column(c == 0 ? -1 : cx + k, c == 0 ? k : cy, X, Y) ? 1u << k : 0u;
      }
    };
    auto halo_col = [&](int k, int c, int& h, int& pos, long& i) {  // h: hyperplane; false: no such column
      h = k - (c == 2 ? 3 : 1);
      pos = c == 0 ? 0 : (c == 1 ? k + 1 : k);
      const bool ok = k < K && ((hmask[c] >> k) & 1u) != 0;
      i = ok ? hbase[c] + (long)k * hstep[c] : 0;
      return ok;
    };
    auto halo_load = [&](int k, V (&v)[NC][2]) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        int h, pos;
        long i;
        halo_col(k, c, h, pos, i);
#pragma unroll
        for (int q = 0; q < 2; ++q) v[c][q] = cload(a.x + i + (64 * q + lane < nz ? 64 * q + lane : 0));
      }
    };
    auto missing = [&](int k, const V (&v)[NC][2]) {
      bool miss = false;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        int h, pos;
        long i;
        if (halo_col(k, c, h, pos, i)) {
#pragma unroll
          for (int q = 0; q < 2; ++q) miss |= B::bits(v[c][q]) == B::sent;
        }
      }
      return __builtin_amdgcn_ballot_w64(miss) != 0;
    };
    auto halo_put = [&](int k, V (&v)[NC][2]) {
      if (missing(k, v)) {
        // fall back behind the producers: wait for the next step's columns
        // too, so that later steps find theirs when they are read ahead
        unsigned spins = 0;
        V w[NC][2];
        do {
          if (++spins >= LGS_SPIN_LIMIT) {
            atomicOr(a.err, 1u);
            break;
          }
          if ((spins & 1023u) == 1023u && (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u))
            break;
          __builtin_amdgcn_s_sleep(1);
          halo_load(k, v);
          halo_load(k + 1, w);
        } while (missing(k, v) || missing(k + 1, w));
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        int h, pos;
        long i;
        if (halo_col(k, c, h, pos, i)) {
#pragma unroll
          for (int q = 0; q < 2; ++q)
            if (64 * q + lane < nz) ringp(h, pos)[64 * q + lane] = v[c][q];
        }
      }
    };
    // the finished column of step k, device-coherently, and its sentinel in `next`
    auto store = [&](int k) {
      int Y;
      if (at_step(k, Y)) {
        const long i = tb + ((Xp - X0) * g.ny + Y) * nz + z;
        cstore(a.x + i, ringp(k, lx + 1)[z]);
        if (a.next) a.next[i] = B::val(B::sent);
      }
    };

    if (wave < npw) {
      LtPoint<PAT, V> p0, p1;
      load(p0, 0);
      load(p1, 1);
      stage(p0, 0);
      __syncthreads();
      auto step = [&](LtPoint<PAT, V>& p, LtPoint<PAT, V>& pn, int k) {
        store(k - 1);
        rhs(p, k);
        __syncthreads();
        load(p, k + 2);
        stage(pn, k + 1);
        __syncthreads();
      };
#pragma unroll 1
      for (int k = 0; k < nsteps; k += 2) {
        step(p0, p1, k);
        if (k + 1 < nsteps) step(p1, p0, k + 1);
      }
      store(nsteps - 1);
    } else if (wave == npw) {
      __builtin_amdgcn_s_setprio(3);
      __syncthreads();
      for (int k = 0; k < nsteps; ++k) {
        __syncthreads();
        solve(k);
        __syncthreads();
      }
    } else {
      halo_plan();
      if (SH) {  // step 0 also reads (-1, -1)
        int X, Y;
        if (column(-1, -1, X, Y)) {
          const long i = ((long)X * g.ny + Y) * nz;
          for (int q = lane; q < nz; q += 64) ringp(-2, 0)[q] = await_value(a.x + i + q, cload(a.x + i + q), a.err);
        }
      }
      halo_load(0, hv);
      halo_put(0, hv);
      halo_load(1, hv);
      __syncthreads();
      for (int k = 0; k < nsteps; ++k) {
        __syncthreads();
        halo_put(k + 1, hv);
        halo_load(k + 2, hv);
        __syncthreads();
      }
    }
  }
  lgs_retire(a.ctr);
}

// Thomas pivots of every z-column (FP64, one thread per column).
__global__ __launch_bounds__(256) void k_tri_factor(Grid g, int slo, int sc, int sup, const double* __restrict__ A,
                                                     double* __restrict__ rden, double* __restrict__ cp,
                                                     unsigned* err) {
  const long col = (long)blockIdx.x * 256 + threadIdx.x;
  if (col >= (long)g.nx * g.ny) return;
  const long N = g.N();
  const long i0 = col * g.nz;
  double cprev = 0.0;
  for (int Z = 0; Z < g.nz; ++Z) {
    const long i = i0 + Z;
    const double az = Z > 0 ? A[(long)slo * N + i] : 0.0;
    const double cz = Z < g.nz - 1 ? A[(long)sup * N + i] : 0.0;
    const double piv = Z == 0 ? A[(long)sc * N + i] : fma(-az, cprev, A[(long)sc * N + i]);
    if (piv == 0.0) atomicOr(err, 2u);
    const double r = 1.0 / piv;
    rden[i] = r;
    cprev = cz * r;
    cp[i] = cprev;
  }
}

template <int PAT, int DIR, class V, bool ZG>
hipError_t launch_lgs_t(const LgsArgs<V>& a, hipStream_t st) {
  const unsigned total = (unsigned)a.ntile;
  if (a.g.nz <= LT_MAX_NZ) {
    const unsigned tgrid = total < (unsigned)LT_MAX_GRID ? total : (unsigned)LT_MAX_GRID;
    const unsigned threads = (unsigned)((a.K * a.g.nz + 63) / 64 + 2) * 64u;
    const size_t smem = ((size_t)7 * a.K * lt_ldp(a.g.nz) + (size_t)4 * (a.K + 1) * lt_rz(a.g.nz)) * sizeof(V);
    hipLaunchKernelGGL((k_lgs_tile<PAT, DIR, V, ZG>), dim3(tgrid), dim3(threads), smem, st, a);
    return hipGetLastError();
  }
  const unsigned grid = total < (unsigned)LGS_MAX_GRID ? total : (unsigned)LGS_MAX_GRID;
  if (a.K != 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_lgs<PAT, DIR, V, ZG>), dim3(grid), dim3(LGS_NT), 4 * sizeof(V) * a.g.nz, st, a);
  return hipGetLastError();
}

template <int PAT, class V>
hipError_t launch_lgs_p(int dir, bool zg, const LgsArgs<V>& a, hipStream_t st) {
  if (dir > 0) return zg ? launch_lgs_t<PAT, 1, V, true>(a, st) : launch_lgs_t<PAT, 1, V, false>(a, st);
  if (zg) return hipErrorInvalidValue;  // the zero-guess sweep is the forward pre-smoother
  return launch_lgs_t<PAT, -1, V, false>(a, st);
}

}  // namespace

// Tile side: a hyperplane of a tile is K columns, at most pts points.
static int lgs_side(const Grid& g, int pts) { return g.nz >= pts ? 1 : (pts / g.nz < 8 ? pts / g.nz : 8); }

static int lgs_tiles(const Grid& g, int pat, int k, std::vector<int>* tmap) {
  const int sh = lgs_cwx(pat) - 1;
  const int ntx = (g.nx + k - 1) / k, nty = (g.ny + sh * (g.nx - 1) + k - 1) / k;
  int n = 0;
  for (int d = 0; d < ntx + nty - 1; ++d) {
    // (only these bx can hold a column: sh*bx <= by <= sh*(bx + 1) + (ny - 1) / k)
    const int b0 = std::max((d - sh - (g.ny - 1) / k) / (1 + sh) - 1, 0), b1 = std::min(d / (1 + sh) + 1, ntx - 1);
    for (int bx = b0; bx <= b1; ++bx) {
      const int by = d - bx;
      if (by < 0 || by >= nty) continue;
      // the tile holds a column if some x of it has y = y' - sh*x in [0, ny)
      bool any = false;
      for (int x = bx * k; x < bx * k + k && x < g.nx && !any; ++x) {
        const int y0 = by * k - sh * x, y1 = y0 + k - 1;
        any = y1 >= 0 && y0 < g.ny;
      }
      if (!any) continue;
      if (tmap) tmap->push_back((bx << 16) | by);
      ++n;
    }
  }
  return n;
}

static int lgs_points(const Grid& g, int vbytes) {
  return g.nz > LT_MAX_NZ ? 1 : (vbytes == 4 ? lt_pts<float>() : lt_pts<double>());
}

int lgs_plan(const Grid& g, int pat, int vbytes, int* K, std::vector<int>* tmap) {
  *K = lgs_side(g, lgs_points(g, vbytes));
  return lgs_tiles(g, pat, *K, tmap);
}

// A tile's entry in the table: bx above bit 16 of a signed word, by below.
bool lgs_ranges_ok(const Grid& g, int pat, int vbytes) {
  const int sh = lgs_cwx(pat) - 1, k = lgs_side(g, lgs_points(g, vbytes));
  return (g.nx - 1) / k < 1 << 15 && ((long)g.ny - 1 + (long)sh * (g.nx - 1)) / k < 1 << 16;
}

// (the smaller tiles of every precision)
int lgs_reserve(const Grid& g, int pat) { return lgs_tiles(g, pat, lgs_side(g, LGS_RESERVE_PTS), nullptr); }

hipError_t launch_tri_factor(int pat, const Grid& g, const double* A, double* rden, double* cp, unsigned* err,
                             hipStream_t st) {
  const int slo = pat_slot(pat, 0, 0, -1), sc = pat_slot(pat, 0, 0, 0), sup = pat_slot(pat, 0, 0, 1);
  if (slo < 0 || sc < 0 || sup < 0) return hipErrorInvalidValue;
  const long ncol = (long)g.nx * g.ny;
  hipLaunchKernelGGL(k_tri_factor, dim3((unsigned)((ncol + 255) / 256)), dim3(256), 0, st, g, slo, sc, sup, A, rden,
                     cp, err);
  return hipGetLastError();
}

template <class V>
hipError_t launch_lgs(int pat, int dir, bool zero_guess, const LgsArgs<V>& a, hipStream_t st) {
  if (a.K < 1 || a.ntile < 1 || !a.tmap || a.g.nz > LGS_MAX_NZ || (!zero_guess && a.uold == nullptr))
    return hipErrorInvalidValue;
  if (pat == 7) return launch_lgs_p<7, V>(dir, zero_guess, a, st);
  if (pat == 19) return launch_lgs_p<19, V>(dir, zero_guess, a, st);
  if (pat == 27) return launch_lgs_p<27, V>(dir, zero_guess, a, st);
  return hipErrorInvalidValue;
}

template hipError_t launch_lgs<double>(int, int, bool, const LgsArgs<double>&, hipStream_t);
template hipError_t launch_lgs<float>(int, int, bool, const LgsArgs<float>&, hipStream_t);

}  // namespace smg
