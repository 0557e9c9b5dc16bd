// Dependence-preserving structured triangular sweep (Sec. 4.4): point
// Gauss-Seidel and the ILU(0) factor solves, computed in exactly the order of
// the sequential lexicographic sweep, so the result equals the serial one.
//
// Row update (T = lower offsets for a forward sweep, upper for a backward one):
//     t = h_i;  for s in T (canonical order): t = fma(-c_s[i], x[i+off_s], t);
//     x_i = t * d_i          (or x_i = t for a unit diagonal)
// Couplings to points outside the grid are stored as zero and their values
// read as zero, so every term is applied unconditionally.
//
// GPU design (replaces the CPU design of the paper, which projects the grid
// onto x-y columns, runs level-scheduled column tasks and synchronises
// threads point-to-point through a shared counter array):
//  * The z-column is the unit.  A workgroup owns a TX x TY tile of columns:
//    tile (X, Y) holds x in [X*TX, X*TX+TX) and y + sh*(x - X*TX) in
//    [Y*TY, Y*TY+TY) (sheared so that no dependence points from a tile to a
//    later one).
//  * Column (lx, ly) of the tile handles point z at step s = z + skew(lx, ly),
//    skew = (wx - sh*wy)*lx + wy*ly + KB with the hyperplane weights
//    (wx, wy, 1) of the pattern; a neighbour at offset (dx, dy, dz) is then
//    handled exactly wx*dx + wy*dy + dz steps away, the same for every
//    column, which is earlier for every lower neighbour.  A backward sweep
//    runs the same tiles and steps in reverse order.  KB pads both ends of
//    the step range so that values referenced at the first and last steps
//    have a step.
//  * A step costs the time a wave needs to issue its instructions (one per
//    four cycles at best) plus one exchange of values through LDS, so the
//    workgroup splits the work by role, each role in waves of its own, and
//    all waves meet at one workgroup barrier per step:
//      - two compute waves, one column per lane: the chain of fmas, the
//        result to LDS, and the packed coefficients (a schedule-ordered copy,
//        16-byte coalesced loads, P steps ahead); no global stores and no
//        waits on memory other than their own coefficient loads;
//      - a halo wave: fetches the values of neighbouring tiles' columns from
//        their strips (below) into the LDS ring;
//      - a load wave: streams the right-hand side into LDS as runs of 16
//        consecutive z per column, two chunks of 16 steps ahead;
//      - a store wave: streams the results out of LDS as runs, one chunk
//        behind;
//      - an export wave: writes the tile's strip.
//    Loads and stores never share a wave: a wave's vector memory operations
//    retire in issue order, so a wave that waits for a load would also wait
//    for every store issued before it, and no more than 63 may be in flight.
//    Values that cross waves move through an LDS ring of 16 steps (the tile's
//    columns plus a halo of neighbouring tiles' columns) and three chunk
//    buffers (one filled, one computed, one drained).
//  * Inactive positions (a column outside the grid, or z outside [0, nz) at
//    that step) have zero coefficients, scaling and right-hand side, so
//    their result is zero without a test as long as every value they read is
//    finite: the LDS is zeroed once per launch.  In a grouped launch the tile
//    before may be another system's, whose values overflowed (a zero
//    coefficient does not stop those), so the ring rows that a tile reads
//    before it writes them are zeroed ahead of it.
//  * Tiles exchange values through strips: per step a tile writes the values
//    of the columns that others read (23 of 128, 30 with 19/27 points) as one
//    contiguous run, device-coherently.  A hyperplane has one step number per
//    tile, so what a tile needs at a step from one neighbour is one step's
//    run of that neighbour: two or three line reads instead of one scattered
//    8-byte access per column, and the results themselves are plain full-line
//    stores.  An entry holds a signalling-NaN sentinel until it is written; a
//    value is ready when it is no longer the sentinel.  Each level has two
//    strip buffers: a sweep uses one and restores the sentinels of the other
//    (the last workgroup switches them), so any sequence of sweeps, in either
//    direction and onto any output, finds its buffer ready.  Forward sweep
//    with 16 x 16 tiles before / after (exports and sentinels in the output,
//    one wave for results and exports -> strips, an export wave; MI355X,
//    FP64): 256^3 7-point 757 -> 383 us, 128^3 27-point 840 -> 641 us,
//    512x512x64 19-point 2662 -> 1846 us; an isolated 7-point tile steps in
//    0.166 instead of 0.283 us (the store wave's limit of 63 stores in flight).
//  * Tiles are 8 columns wide in x.  A CU streams a tile's coefficients at
//    40-70 GB/s whatever the prefetch depth, and LDS reads and 16-byte loads
//    of four compute waves queue up in each step, so half the columns per CU
//    nearly halve a step (27-point FP64 0.335 -> 0.18, FP32 0.22 -> 0.145,
//    7-point 0.166 -> 0.124 us) while the hand-offs only grow by half.
//    Forward sweep, 16 / 8 / 4 columns wide: 128^3 27-point FP64 638 / 396 /
//    347 us, FP32 260 / 213 / 283 us; 64^3 FP64 197 / 132 / 164 us; 256^3
//    7-point 384 / 330 / 426 us; 512x512x64 19-point 1844 / 1650 / 2114 us.
//  * A halo wave that finds a value not yet written waits for the values
//    AHEAD steps further on and refetches its prefetched values with them:
//    the tile then runs far enough behind its producer that later prefetches
//    find their values written, instead of paying one coherent round trip
//    per step.
//  * Tiles are handed out by an atomic ticket in dependence order, so a
//    persistent grid of any size always makes progress.  Waits are bounded
//    by a watchdog that raises an error flag instead of hanging.
//  * All per-point accesses use buffer instructions; positions without a
//    point use an offset outside the buffer, for which loads return zero
//    and stores are dropped.
#include "smg_common.h"
#include "smg_group.h"
#include "smg_kernels.h"
#include "smg_sweep.h"

namespace smg {

constexpr int WF_HIST = 16;                  // LDS ring rows (steps)
constexpr int WF_CH = 16;                    // steps per chunk of right-hand side / results
constexpr int WF_NB = 3;                     // chunk buffers: filled, computed, drained
constexpr int WF_NL = WF_TX * WF_TY;         // compute lanes (columns) per tile
constexpr int WF_NCW = WF_NL / 64;           // compute waves
constexpr int WF_THREADS = 64 * (WF_NCW + 4);  // ... and a halo, a load, a store and an export wave
constexpr int WF_NH = 20 + 2 * WF_TX;        // halo slots around a tile
constexpr int WF_GRP = WF_NL * WF_CH / 64;   // column-run groups per chunk (4 columns x 16 steps)
constexpr int WF_GPS = WF_GRP / WF_CH;       // groups moved per step
constexpr int WF_RW = WF_NL + WF_NH + 1;     // ring row length (padded)
constexpr int WF_HRW = WF_NL + 1;            // chunk buffer row length (padded)
#ifndef WF_LAG_EXTRA
#define WF_LAG_EXTRA 2
#endif
#ifndef WF_PH
#define WF_PH 4
#endif

// Neighbour columns holding lower neighbours (forward-frame offsets); a
// backward sweep uses the negated offsets.
__host__ __device__ constexpr int col_dx(int c) { return c == 3 ? 0 : -1; }
__host__ __device__ constexpr int col_dy(int c) { return c == 3 ? -1 : c - 1; }
__host__ __device__ constexpr bool col_used(int pat, int c) {
  return pat_has(pat, col_dx(c), col_dy(c), -1) || pat_has(pat, col_dx(c), col_dy(c), 0) ||
         pat_has(pat, col_dx(c), col_dy(c), 1);
}
__host__ __device__ constexpr int col_of(int dx, int dy) {
  return dx == -1 ? dy + 1 : (dy == -1 ? 3 : -1);
}

// Largest step distance of a lower neighbour: max over lower offsets of
// -(wx*dx + wy*dy + dz).
__host__ __device__ constexpr int wf_kb(int pat) {
  int m = 0;
  for (int s = 0; s < pat / 2; ++s) {
    const int d = -(hp_wx(pat) * pat_off(pat, s, 0) + hp_wy(pat) * pat_off(pat, s, 1) + pat_off(pat, s, 2));
    m = d > m ? d : m;
  }
  return m;
}

// Term m of a sweep's triangle (canonical order): step distance of its
// neighbour (in [-KB, -1]) and, leading terms only, how many have a value at
// least two steps old.
__host__ __device__ constexpr int wf_back(int pat, int dir, int m) {
  const int so = dir > 0 ? m : pat / 2 + 1 + m;
  return dir * (hp_wx(pat) * pat_off(pat, so, 0) + hp_wy(pat) * pat_off(pat, so, 1) + pat_off(pat, so, 2));
}
__host__ __device__ constexpr int wf_prefix(int pat, int dir) {
  int n = 0;
  while (n < pat / 2 && wf_back(pat, dir, n) <= -2) ++n;
  return n;
}

// 16-byte packs per point and direction: the pat/2 coefficients of the
// sweep's triangle followed (except for FP16 storage, which keeps it apart)
// by the diagonal scaling.
__host__ __device__ constexpr int wf_npk(int pat, int ebytes) {
  return (pat / 2 + (ebytes == 2 ? 0 : 1) + 16 / ebytes - 1) / (16 / ebytes);
}
// FP16 storage: do the position's FP32 {row scale, diagonal scaling} fit in
// the last two words of its packs (after the pattern's lower halves)?  Then a
// step loads them with the coefficients (7- and 19-point: one load per step
// instead of two); otherwise (27-point) they come from a separate array.
__host__ __device__ constexpr bool wf_sd_in_pack(int pat) { return pat / 2 + 4 <= 8 * wf_npk(pat, 2); }

// Does the last pack have a word that no step uses?
__host__ __device__ constexpr bool wf_loose_pack(int pat, int ebytes) {
  return ebytes == 2 ? pat != 7 : (pat / 2 + 1) % (16 / ebytes) != 0;
}

// Tiles of tx x 16 columns.
static void wf_tile(const Grid& g, int pat, WfTiling* t, int shape, int tx) {
  // Default: tiles are sheared (y + x offset) when a lower neighbour column
  // lies at (x-1, y+1) (19- and 27-point patterns), so that every dependence
  // points to an earlier tile in x and y; otherwise, and when a single tile
  // row covers y, plain rectangles, which give fewer tile hand-offs on the
  // critical path.  Shears are valid for every pattern (a point's step is its
  // hyperplane index minus a per-tile offset either way).  Rectangles are not
  // for 19/27-point sweeps with more than one tile row: column (x, y) of a
  // tile's top row then reads (x-1, y+1) in the tile above, which reads the
  // tile below through (x, y-1), and two tiles waiting on each other stall
  // (retile_level refuses that case).  shape 1 / 2 forces sheared /
  // rectangular tiles.
  t->sh = shape == 1 ? 1 : (shape == 2 ? 0 : ((pat == 7 || g.ny <= WF_TY) ? 0 : 1));
  t->ntx = (g.nx + tx - 1) / tx;
  t->nty = (g.ny + t->sh * (tx - 1) + WF_TY - 1) / WF_TY;
  const int kb = wf_kb(pat);
  t->ns = g.nz + (hp_wx(pat) - t->sh * hp_wy(pat)) * (tx - 1) + hp_wy(pat) * (WF_TY - 1) + 2 * kb;
  t->nsk = (long)t->ntx * t->nty * t->ns * tx * WF_TY;
}

void wf_tiling(const Grid& g, int pat, WfTiling* t, int shape) { wf_tile(g, pat, t, shape, WF_TX); }

long wf_reserve(const Grid& g, int pat, int shape) {
  WfTiling t;
  wf_tile(g, pat, &t, shape, 16);
  return t.nsk;
}

int wf_pack_count(int pat, int ebytes) { return wf_npk(pat, ebytes); }

bool wf_ranges_ok(const Grid& g, const WfTiling& t, int pat, int vbytes, int ebytes) {
  const double vec = (double)(WF_TX + 2) * g.ny * g.nz * vbytes;
  const double tile = (double)t.ns * wf_npk(pat, ebytes) * WF_NL * 16;
  return vec < 2147483647.0 && tile < 2147483647.0;
}

// Halo slot of column (qx, qy) relative to a tile (outside [0,TX) x [0,TY)).
// In the forward frame (a backward sweep mirrors both axes) these are the
// column x-1 with y in [-2, TY+2), the row y = -1 and one second row: y = -2
// (sheared tiles) or y = TY (rectangles, whose lower neighbours reach
// (x-1, y+1)).
__host__ __device__ constexpr int wf_halo_slot(int dir, int qx, int qy) {
  const int fx = dir > 0 ? qx : WF_TX - 1 - qx, fy = dir > 0 ? qy : WF_TY - 1 - qy;
  return fx < 0 ? fy + 2 : (fy == -1 ? 20 + fx : 20 + WF_TX + fx);
}
// Forward-frame position of slot t.
__device__ inline void wf_halo_pos(int sh, int t, int* fx, int* fy) {
  *fx = t < 20 ? -1 : (t < 20 + WF_TX ? t - 20 : t - 20 - WF_TX);
  *fy = t < 20 ? t - 2 : (t < 20 + WF_TX ? -1 : (sh ? -2 : WF_TY));
}

// Export strips.  Per step a tile publishes the values of the columns that
// other tiles read as one contiguous run of wf_es entries: the 16 columns
// lx = TX-1, then the TX columns ly = TY-1, then (19/27 points) the TX columns
// of the second row (ly = TY-2 of sheared tiles, ly = 0 of rectangles), all in
// the forward frame.  Entry e of step s of a tile is at
// ((tile*NS + s)*wf_es + e).
__host__ __device__ constexpr int wf_es(int pat) { return WF_TY + (pat == 7 ? WF_TX : 2 * WF_TX); }
__device__ inline int wf_export_lane(int dir, int sh, int e) {
  int lx = e < WF_TY ? WF_TX - 1 : (e - WF_TY) % WF_TX;
  int ly = e < WF_TY ? e : (e < WF_TY + WF_TX ? WF_TY - 1 : (sh ? WF_TY - 2 : 0));
  if (dir < 0) {
    lx = WF_TX - 1 - lx;
    ly = WF_TY - 1 - ly;
  }
  return lx * WF_TY + ly;
}
long wf_strip_elems(const WfTiling& t, int pat) { return (long)t.ntx * t.nty * t.ns * wf_es(pat); }

// Is halo column (qx, qy) a neighbour column of some lane of the tile in a
// sweep of direction dir?
__device__ inline bool wf_halo_used(int pat, int dir, int sh, int qx, int qy) {
  for (int c = 0; c < 4; ++c) {
    if (!col_used(pat, c)) continue;
    const int cx = dir * col_dx(c), cy = dir * col_dy(c);
    const int lx = qx - cx, ly = qy - cy - sh * cx;
    if (lx >= 0 && lx < WF_TX && ly >= 0 && ly < WF_TY) return true;
  }
  return false;
}

// Storage element traits: arithmetic type V, elements per 16-byte pack K,
// and element m of a run of packs.
template <class E>
struct WfE;
template <>
struct WfE<double> {
  using V = double;
  static constexpr int K = 2;
  static constexpr bool HALF = false;
  __device__ static double get(const u32x4* pk, int m) {
    const u32x4 w = pk[m / 2];
    return m % 2 == 0 ? __builtin_bit_cast(double, u32x2{w.x, w.y}) : __builtin_bit_cast(double, u32x2{w.z, w.w});
  }
};
template <>
struct WfE<float> {
  using V = float;
  static constexpr int K = 4;
  static constexpr bool HALF = false;
  __device__ static float get(const u32x4* pk, int m) { return __uint_as_float(pk[m / 4][m % 4]); }
};
template <>
struct WfE<__half> {
  using V = float;
  static constexpr int K = 8;
  static constexpr bool HALF = true;
  __device__ static float get(const u32x4* pk, int m) {
    const unsigned w = pk[m / 8][(m % 8) / 2];
    return __half2float(__ushort_as_half((unsigned short)(m % 2 == 0 ? (w & 0xffffu) : (w >> 16))));
  }
  // the row-scaled coefficient float(h_m) * sc in one instruction
  __device__ static float scaled(const u32x4* pk, int m, float sc) {
    const unsigned w = pk[m / 8][(m % 8) / 2];
    return m % 2 == 0 ? half_times<0>(w, sc) : half_times<1>(w, sc);
  }
};

// Geometry of one tile shared by all roles.
struct WfGeo {
  int X, Y, sh, NS, nsteps;
  int p0;             // first x plane of the vector buffers
  unsigned vbytes;    // bytes of the vector buffers (planes p0 .. p1-1)
  long vb;            // element offset of plane p0
  bool full;          // every column of the tile lies in the grid
};

template <class V>
__device__ inline WfGeo wf_geo(const WfArgs<V>& a, unsigned tile) {
  WfGeo q;
  q.X = (int)(tile / (unsigned)a.t.nty);
  q.Y = (int)(tile % (unsigned)a.t.nty);
  q.sh = a.t.sh;
  q.NS = a.t.ns;
  q.nsteps = (q.NS + WF_CH - 1) / WF_CH * WF_CH;
  q.p0 = q.X * WF_TX > 0 ? q.X * WF_TX - 1 : 0;
  const int p1 = q.X * WF_TX + WF_TX + 1 < a.g.nx ? q.X * WF_TX + WF_TX + 1 : a.g.nx;
  const long pl = (long)a.g.ny * a.g.nz;
  q.vbytes = (unsigned)((p1 - q.p0) * pl * (long)sizeof(V));
  q.vb = q.p0 * pl;
  const int y0 = q.Y * WF_TY;
  q.full = q.X * WF_TX + WF_TX <= a.g.nx && y0 - q.sh * (WF_TX - 1) >= 0 && y0 + WF_TY <= a.g.ny;
  return q;
}

template <int DIR>
__device__ inline int wf_step(int NS, int k) {
  return DIR > 0 ? k : NS - 1 - k;
}

// ---- compute role (the first two waves) ---------------------------------------
template <int PAT, int DIR, int P, class E, bool UNITD>
__device__ __forceinline__ void wf_compute(const WfArgs<typename WfVal<E>::V>& a, const WfGeo& q, unsigned tile,
                                           typename WfVal<E>::V* ring, typename WfVal<E>::V* hbuf) {
  using T = WfE<E>;
  using V = typename T::V;
  constexpr int C = PAT / 2;
  constexpr int NT = PAT / 2;
  constexpr int WX = hp_wx(PAT), WY = hp_wy(PAT);
  constexpr int NPK = wf_npk(PAT, sizeof(E));
  constexpr unsigned PACKB = WF_NL * 16u;
  static_assert(WF_HIST % P == 0 && WF_HIST > wf_kb(PAT) + 1, "ring too short");
  const int tid = threadIdx.x;
  const int lx = tid / WF_TY, ly = tid % WF_TY;
  const int NS = q.NS;

  // LDS index of each neighbour column within a ring row (offsets mirrored
  // for a backward sweep): a lane of this tile or a halo slot
  int nidx[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int cx = DIR * col_dx(c), cy = DIR * col_dy(c);
    const int qx = lx + cx, qy = ly + cy + q.sh * cx;
    const bool in = qx >= 0 && qx < WF_TX && qy >= 0 && qy < WF_TY;
    nidx[c] = !col_used(PAT, c) ? 0 : (in ? qx * WF_TY + qy : WF_NL + wf_halo_slot(DIR, qx, qy));
  }
  const unsigned tbytes = (unsigned)NS * NPK * PACKB;
  const auto rp = wf_rsrc((const char*)a.pk + (size_t)tile * tbytes, tbytes);
  const unsigned sdbytes = T::HALF ? (unsigned)NS * WF_NL * 8u : 0u;
  const auto rs = wf_rsrc(T::HALF ? (const char*)a.sd + (size_t)tile * sdbytes : (const char*)a.pk, sdbytes);

  // Positions without a point (z outside [0, nz) or the column outside the
  // grid) take an offset outside the buffer: their coefficients read as zero
  // without a memory access, so the copy's padding costs no traffic.
  const int skew = (WX - q.sh * WY) * lx + WY * ly + wf_kb(PAT);
  const int xt = q.X * WF_TX + lx, yt = q.Y * WF_TY + ly - q.sh * lx;
  const unsigned zlim = xt < a.g.nx && yt >= 0 && yt < a.g.ny ? (unsigned)a.g.nz : 0u;
  u32x4 cf[P][NPK];
  u32x2 sdv[P];
  // Offsets of step k's packs; pack p (and, with the last, the FP16 scalars)
  // into slot j.
  struct Po {
    unsigned so, vo, ss, vs;
  };
  auto pack_off = [&](int k) {
    const int s = wf_step<DIR>(NS, k);
    const bool sin = s >= 0 && s < NS;
    const bool pt = (unsigned)(s - skew) < zlim;
    return Po{sin ? (unsigned)s * (NPK * PACKB) : WF_OOB, pt ? tid * 16u : WF_OOB,
              sin ? (unsigned)s * (WF_NL * 8u) : WF_OOB, pt ? tid * 8u : WF_OOB};
  };
  auto pack_load = [&](const Po& o, int j, int p) {
    cf[j][p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, o.vo, o.so + p * PACKB, 0));
    if (T::HALF && !wf_sd_in_pack(PAT) && p == NPK - 1)
      sdv[j] = __builtin_amdgcn_raw_buffer_load_b64(rs, o.vs, o.ss, 0);
  };
  constexpr int NPRE = wf_prefix(PAT, DIR);
#pragma unroll
  for (int j = 0; j < P; ++j) {
    // (step 0 has no points: its prefix is skipped, so slot 0 starts with the
    // prefix packs of step P)
    const Po o = pack_off(j), on = pack_off(j + P);
#pragma unroll
    for (int p = 0; p < NPK; ++p) pack_load(j == 0 && p < NPRE / T::K ? on : o, j, p);
  }
  // A step's critical path is: barrier, LDS reads, chain of fmas, LDS write,
  // barrier.  So a step reads after its barrier only the values of the step
  // before (back == -1); older ones were read in the step before, and the
  // leading terms made of older ones (8 of 13 forward, 27-point) are already
  // summed.  Each step then prepares the next one behind its own LDS write.
  constexpr bool SDP = T::HALF && wf_sd_in_pack(PAT);
  V own_prev = V(0), tp = V(0);
  V ve[NT];  // values at least two steps old of the current step's terms
#pragma unroll
  for (int m = 0; m < NT; ++m) ve[m] = V(0);
  __syncthreads();  // prologue: the first chunk is in LDS
  tp = hbuf[tid];   // (the first step's coefficients are zero)

  for (int k0 = 0; k0 < q.nsteps; k0 += WF_HIST) {
    V* hb = hbuf + ((k0 / WF_CH) % WF_NB) * (WF_CH * WF_HRW) + tid;
    const V* hbn = hbuf + ((k0 / WF_CH + 1) % WF_NB) * (WF_CH * WF_HRW) + tid;
#pragma unroll
    for (int j = 0; j < WF_HIST; ++j) {
      const int jp = j % P, jn = (j + 1) % P;
      auto ring_value = [&](int m, int step) {
        const int so = DIR > 0 ? m : C + 1 + m;
        const int c = col_of(DIR * pat_off(PAT, so, 0), DIR * pat_off(PAT, so, 1));
        return ring[((step + wf_back(PAT, DIR, m) + WF_HIST) % WF_HIST) * WF_RW + nidx[c < 0 ? 0 : c]];
      };
      auto own = [](int m) {
        const int so = DIR > 0 ? m : C + 1 + m;
        return pat_off(PAT, so, 0) == 0 && pat_off(PAT, so, 1) == 0;
      };
      auto coeff = [&](int slot, int m) {
        if constexpr (T::HALF)
          return T::scaled(cf[slot], m, __uint_as_float(SDP ? cf[slot][NPK - 1][2] : sdv[slot].x));
        else
          return T::get(cf[slot], m);
      };
      V val[NT], vn[NT];
#pragma unroll
      for (int m = 0; m < NT; ++m)
        val[m] = wf_back(PAT, DIR, m) < -1 ? ve[m] : (own(m) ? own_prev : ring_value(m, j));
#pragma unroll
      for (int m = 0; m < NT; ++m)
        if (wf_back(PAT, DIR, m) < -1) vn[m] = ring_value(m, j + 1);
      const V hn = j + 1 < WF_HIST ? hb[(j + 1) * WF_HRW] : hbn[0];
      __builtin_amdgcn_sched_barrier(0);
      V t = tp;
      const Po po = pack_off(k0 + j + P);
#pragma unroll
      for (int m = NPRE; m < NT; ++m) {
        t = fma(-coeff(jp, m), val[m], t);
        // without a prefix the refilling loads go between the fmas
        if (NPRE == 0 && (m + 1) % T::K == 0 && m / T::K < NPK - 1) {
          __builtin_amdgcn_sched_barrier(0);
          pack_load(po, jp, m / T::K);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      const V dv = T::HALF ? __uint_as_float(SDP ? cf[jp][NPK - 1][3] : sdv[jp].y) : T::get(cf[jp], NT);
      const V xv = UNITD ? t : t * dv;
      // words of the last pack without an entry stay live until here: reused
      // as temporaries they would make their writer wait for every load in
      // flight (27-point FP32: 0.246 instead of 0.15 us per step)
      // (a unit diagonal leaves the scaling's words unused: 512x512x64 19-point
      // FP64 L solve 2952 -> 1685 us)
      if constexpr (UNITD || wf_loose_pack(PAT, sizeof(E))) asm volatile("" : : "v"(cf[jp][NPK - 1]));
      own_prev = xv;
      ring[j * WF_RW + tid] = xv;
      hb[j * WF_HRW] = xv;
      __builtin_amdgcn_sched_barrier(0);
      // refill the packs that were used for the last time (those of the prefix
      // are refilled below, one step earlier)
      constexpr int DONE = NPRE == 0 ? (NT / T::K < NPK - 1 ? NT / T::K : NPK - 1) : NPRE / T::K;
#pragma unroll
      for (int p = DONE; p < NPK; ++p) pack_load(po, jp, p);
      tp = hn;
      const Po pn = pack_off(k0 + j + 1 + P);
#pragma unroll
      for (int m = 0; m < NPRE; ++m) {
        tp = fma(-coeff(jn, m), vn[m], tp);
        if ((m + 1) % T::K == 0 && m / T::K < NPK - 1) {
          __builtin_amdgcn_sched_barrier(0);
          pack_load(pn, jn, m / T::K);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int m = 0; m < NT; ++m)
        if (wf_back(PAT, DIR, m) < -1) ve[m] = vn[m];
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
    }
  }
  __syncthreads();  // tail: the last chunk is drained and the last step exported
  __syncthreads();
}

// ---- halo role ----------------------------------------------------------------
template <int PAT, int DIR, class V>
__device__ __forceinline__ void wf_halo(const WfArgs<V>& a, const WfGeo& q, const V* strip, V* ring, unsigned* err) {
  using B = VBits<V>;
  constexpr int WX = hp_wx(PAT), WY = hp_wy(PAT), ES = wf_es(PAT);
  constexpr int PH = WF_PH;
  constexpr int AHEAD = PH + WF_LAG_EXTRA;  // steps a stalled tile falls back behind its producer
  static_assert(WF_HIST % PH == 0 && PH >= 2, "halo prefetch distance");
  const int t = threadIdx.x - WF_NL;
  const int NS = q.NS;

  // Halo slot t: the producing tile, its export entry and the distance dk
  // between the producer's step and this tile's (a hyperplane has one step
  // number per tile).
  int fx = 0, fy = 0;
  bool role = false;
  if (t < WF_NH) {
    wf_halo_pos(q.sh, t, &fx, &fy);
    role = wf_halo_used(PAT, DIR, q.sh, DIR > 0 ? fx : WF_TX - 1 - fx, DIR > 0 ? fy : WF_TY - 1 - fy);
  }
  const int ax = fx < 0 ? 1 : 0;
  const int fyt = fy + (ax ? WF_TX * q.sh : 0) + 2 * WF_TY;  // >= 0
  const int dyf = fyt / WF_TY - 2, lyf = fyt % WF_TY, lxf = ax ? WF_TX - 1 : fx;
  const int PX = q.X - DIR * ax, PY = q.Y + DIR * dyf;
  const bool have = role && PX >= 0 && PX < a.t.ntx && PY >= 0 && PY < a.t.nty;
  const int dk = DIR * (WX * WF_TX * ax - WY * WF_TY * dyf);
  const int e = lxf == WF_TX - 1 ? lyf : (lyf == WF_TY - 1 ? WF_TY + lxf : WF_TY + WF_TX + lxf);
  const V* hp = have ? strip + (((long)PX * a.t.nty + PY) * NS) * ES + e : strip;
  const int es = have ? ES : 0;

  // does step k have a value, and its address (clamped to the producer's
  // steps, so that every load is unconditional)
  auto valid = [&](int k) {
    const int s = wf_step<DIR>(NS, k), sp = s + dk;
    return have && s >= 0 && s < NS && sp >= 0 && sp < NS;
  };
  auto fetch = [&](int k) {
    int sp = wf_step<DIR>(NS, k) + dk;
    sp = sp < 0 ? 0 : (sp >= NS ? NS - 1 : sp);
    return wf_coherent_load(hp + (long)sp * es);
  };
  V hb[PH];
  // halo values of step k (slot j): wait for any that is still the sentinel,
  // then publish them in ring row k
  auto put = [&](int k, int j) {
    const bool ok = valid(k);
    if (__builtin_amdgcn_ballot_w64(ok && B::bits(hb[j]) == B::sent) != 0) {
      // fall back behind the producer: wait until the values AHEAD steps on
      // are there, and with them this step's and the prefetched ones
      unsigned spins = 0;
      for (;;) {
        const V far = fetch(k + AHEAD);
#pragma unroll
        for (int d = 0; d < PH; ++d) hb[(j + d) % PH] = fetch(k + d);
        const bool miss = (ok && B::bits(hb[j]) == B::sent) || (have && B::bits(far) == B::sent);
        if (__builtin_amdgcn_ballot_w64(miss) == 0) break;
        if (++spins >= WF_SPIN_LIMIT) {
          atomicOr(err, 1u);
          break;
        }
        // once any wait has timed out, stop waiting anywhere
        if ((spins & 1023u) == 1023u && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u)) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (role) ring[(k % WF_HIST) * WF_RW + WF_NL + t] = ok ? hb[j] : V(0);
  };
#pragma unroll
  for (int j = 0; j < PH; ++j) hb[j] = fetch(j);
  __syncthreads();  // prologue

  for (int k0 = 0; k0 < q.nsteps; k0 += PH) {
#pragma unroll
    for (int j = 0; j < PH; ++j) {
      put(k0 + j, j);
      hb[j] = fetch(k0 + j + PH);
      __syncthreads();
    }
  }
  __syncthreads();
  __syncthreads();
}

// ---- column runs (load and store roles) --------------------------------------
// Group r (r = 4 lx + g) of a chunk moves columns 4r + cq (cq = lane / 16), steps m = lane %
// 16 of the chunk: each column's 16 consecutive z values are one coalesced run.
// Per chunk a lane forms its base offsets once, per step the step's bases; a
// group then adds a uniform term.  The bases pass through wf_keep, which the
// compiler may not move across the step's memory operations, so that it does
// not compute every step's offsets ahead (they would hold dozens of
// registers for the whole chunk or sweep).
template <int PAT, int DIR, class V>
struct WfRuns {
  static constexpr int WX = hp_wx(PAT), WY = hp_wy(PAT), KB = wf_kb(PAT);
  int cq, m;
  int lds;        // LDS index of (step m, column cq) within a chunk buffer
  int a0;         // element offset of column cq of group 0 minus its skew
  int y0;         // y of column cq of group 0
  int skq;        // skew of column cq of group 0
  int gx, gy;     // element offset steps per group row (r / 4) and per group (r % 4)
  int sx;         // skew step per group row
  int nx;
  __device__ void init(const WfArgs<V>& a, const WfGeo& q, int lane) {
    nx = a.g.nx;
    cq = lane / 16;
    m = lane % 16;
    lds = m * WF_HRW + cq;
    const int ny = a.g.ny, nz = a.g.nz;
    skq = WY * cq + KB;
    y0 = q.Y * WF_TY + cq;
    a0 = ((q.X * WF_TX - q.p0) * ny + y0) * nz - skq;
    sx = WX - q.sh * WY;
    gx = (ny - q.sh) * nz - sx;
    gy = 4 * (nz - WY);
    vin = (unsigned)(cq * (nz - WY) + (DIR > 0 ? m : WF_CH - 1 - m)) * (unsigned)sizeof(V);
    u0 = ((q.X * WF_TX - q.p0) * ny + q.Y * WF_TY) * nz - KB;
  }
  // Per-chunk bases of this lane's step s of the chunk.
  struct Base {
    int e;    // element offset of group 0
    int z;    // z of group 0
    int u;    // inner chunks: uniform element offset of group 0
    int gx, gy, sx;
  };
  __device__ Base base(const WfGeo& q, int c) const {
    const int s = wf_step<DIR>(q.NS, c * WF_CH + m), lo = wf_step<DIR>(q.NS, c * WF_CH + (DIR > 0 ? 0 : WF_CH - 1));
    return Base{wf_keep(a0 + s), wf_keep(s - skq), u0 + lo, wf_keep_s(gx), wf_keep_s(gy), wf_keep_s(sx)};
  }
  // Per-step bases: the groups moved at one step of a chunk share a column
  // row lx.
  struct Step {
    int e, z, y, lx;
  };
  __device__ Step step(const Base& b, const WfGeo& q, int lx) const {
    // a column row beyond the grid in x takes y = -1 - 16 (outside for every group)
    const int y = q.X * WF_TX + lx < nx ? y0 - q.sh * lx : -WF_TY - 1;
    return Step{wf_keep(b.e + lx * b.gx), wf_keep(b.z - lx * b.sx), wf_keep(y), lx};
  }
  // Offsets of the groups moved at step j of a chunk (GPS*j ..; in: the chunk
  // is inner), vector and scalar parts.
  struct Offs {
    unsigned v[WF_GPS], s[WF_GPS];
  };
  __device__ Offs offs(const WfArgs<V>& a, const WfGeo& q, const Base& b, int j, bool in) const {
    Offs o;
    const int lx = j * WF_GPS / 4, g0 = j * WF_GPS % 4;
    if (in) {
      const int us = wf_keep_s((b.u + lx * b.gx) * (int)sizeof(V));
#pragma unroll
      for (int g = 0; g < WF_GPS; ++g) {
        o.v[g] = vin;
        o.s[g] = (unsigned)(us + (g0 + g) * b.gy * (int)sizeof(V));
      }
    } else {
      const Step t = step(b, q, lx);
#pragma unroll
      for (int g = 0; g < WF_GPS; ++g) {
        o.v[g] = off_any(a, q, b, t, g0 + g);
        o.s[g] = 0u;
      }
    }
    return o;
  }
  // byte offset of group 4*lx + g with every position in the grid
  __device__ static unsigned off_in(const Base& b, const Step& t, int g) {
    return (unsigned)(t.e + g * b.gy) * (unsigned)sizeof(V);
  }
  // Chunks whose 128 x 16 positions are all points (a full tile, away from
  // both ends of its columns): one lane offset for the whole tile plus a
  // uniform byte offset per group, so a group costs no vector arithmetic.
  unsigned vin;          // lane part
  int u0;                // uniform part of group 0 at step 0 (elements)
  __device__ bool inner(const WfArgs<V>& a, const WfGeo& q, int c) const {
    const int lo = wf_step<DIR>(q.NS, c * WF_CH + (DIR > 0 ? 0 : WF_CH - 1));  // steps [lo, lo + WF_CH)
    return q.full && lo >= KB + sx * (WF_TX - 1) + WY * (WF_TY - 1) && lo + WF_CH - 1 - KB < a.g.nz;
  }
  // byte offset of group 4*lx + g, or WF_OOB where the position is outside the grid
  __device__ static unsigned off_any(const WfArgs<V>& a, const WfGeo& q, const Base& b, const Step& t, int g) {
    const int yt = t.y + 4 * g;
    const int z = t.z - 4 * WY * g;
    const bool ok = (unsigned)yt < (unsigned)a.g.ny && (unsigned)z < (unsigned)a.g.nz;
    return ok ? off_in(b, t, g) : WF_OOB;
  }
};

// ---- load role: right-hand side, two chunks ahead --------------------
template <int PAT, int DIR, class V>
__device__ __forceinline__ void wf_load(const WfArgs<V>& a, const WfGeo& q, V* hbuf) {
  using RU = WfRuns<PAT, DIR, V>;
  const int lane = threadIdx.x - WF_NL - 64;
  RU R;
  R.init(a, q, lane);
  const auto rh = wf_rsrc(a.h + q.vb, q.vbytes);
  V reg[WF_GRP];
  // Per step j of a chunk: the registers of the step's groups (a chunk's
  // runs) go to the chunk buffer hb, then take the runs of chunk c.
  auto advance = [&](V* hb, int c, bool sync) {
    const typename RU::Base b = R.base(q, c);
    const bool in = R.inner(a, q, c);
#pragma unroll
    for (int j = 0; j < WF_HIST; ++j) {
      // (the last two rows together: the compute waves read a chunk's first
      // step one step ahead)
#pragma unroll
      for (int i = j < WF_HIST - 2 ? j : WF_HIST - 2; i < WF_HIST && i <= (j < WF_HIST - 2 ? j : WF_HIST - 1); ++i) {
        if (j == WF_HIST - 1) break;
#pragma unroll
        for (int g = 0; g < WF_GPS; ++g) hb[4 * (i * WF_GPS + g)] = reg[i * WF_GPS + g];
        const typename RU::Offs o = R.offs(a, q, b, i, in);
#pragma unroll
        for (int g = 0; g < WF_GPS; ++g) reg[i * WF_GPS + g] = bld<V, 0>(rh, o.v[g], o.s[g]);
      }
      if (sync)
        __syncthreads();
      else
        __builtin_amdgcn_sched_barrier(0);  // keep the refill behind this step's LDS writes
    }
  };
  // prologue: chunk 0 into buffer 0, chunk 1 into the registers
  {
    const typename RU::Base b = R.base(q, 0);
#pragma unroll
    for (int j = 0; j < WF_HIST; ++j) {
      const typename RU::Offs o = R.offs(a, q, b, j, false);
#pragma unroll
      for (int g = 0; g < WF_GPS; ++g) reg[j * WF_GPS + g] = bld<V, 0>(rh, o.v[g], o.s[g]);
    }
  }
  advance(hbuf + R.lds, 1, false);
  __syncthreads();

  for (int k0 = 0; k0 < q.nsteps; k0 += WF_HIST) {
    const int c = k0 / WF_CH;
    // chunk c+1's groups into LDS, then chunk c+2's into the registers freed
    advance(hbuf + ((c + 1) % WF_NB) * (WF_CH * WF_HRW) + R.lds, c + 2, true);
  }
  __syncthreads();
  __syncthreads();
}

// ---- store role: results, one chunk behind ---------------------------
template <int PAT, int DIR, class V>
__device__ __forceinline__ void wf_store(const WfArgs<V>& a, const WfGeo& q, V* hbuf) {
  using RU = WfRuns<PAT, DIR, V>;
  const int lane = threadIdx.x - WF_NL - 128;
  RU R;
  R.init(a, q, lane);
  const auto rx = wf_rsrc(a.x + q.vb, q.vbytes);
  auto chunk = [&](int c, bool sync) {
    const V* hb = hbuf + (c % WF_NB) * (WF_CH * WF_HRW) + R.lds;
    const typename RU::Base b = R.base(q, c);
    const bool in = R.inner(a, q, c);
#pragma unroll
    for (int j = 0; j < WF_HIST; ++j) {
      const typename RU::Offs o = R.offs(a, q, b, j, in);
#pragma unroll
      for (int g = 0; g < WF_GPS; ++g) bst<0>(hb[4 * (j * WF_GPS + g)], rx, o.v[g], o.s[g]);
      if (sync) __syncthreads();
    }
  };
  __syncthreads();  // prologue
#pragma unroll 1
  for (int j = 0; j < WF_HIST; ++j) __syncthreads();
  for (int k0 = WF_HIST; k0 < q.nsteps; k0 += WF_HIST) chunk(k0 / WF_CH - 1, true);
  __syncthreads();
  chunk(q.nsteps / WF_CH - 1, false);
  __syncthreads();
}

// ---- export role: the columns other tiles read -----------------------
// One step after a value is computed it goes to this sweep's strip buffer
// (device-coherently); the other buffer's entry gets the sentinel for the next
// sweep on the level.
template <int PAT, int DIR, class V>
__device__ __forceinline__ void wf_export(const WfArgs<V>& a, const WfGeo& q, unsigned tile, V* strip, V* other,
                                          const V* ring) {
  using B = VBits<V>;
  constexpr int ES = wf_es(PAT);
  const int e = threadIdx.x - WF_NL - 192;
  const bool role = e < ES;
  const int el = role ? wf_export_lane(DIR, q.sh, e) : 0;
  const long base = (long)tile * q.NS * ES + e;
  auto step = [&](int k) {
    if (role && k >= 0 && k < q.NS) {
      const long o = base + (long)wf_step<DIR>(q.NS, k) * ES;
      wf_coherent_store(strip + o, ring[(k % WF_HIST) * WF_RW + el]);
      other[o] = B::val(B::sent);
    }
  };
  __syncthreads();  // prologue
  for (int k = 0; k < q.nsteps; ++k) {
    step(k - 1);
    __syncthreads();
  }
  __syncthreads();
  step(q.nsteps - 1);
  __syncthreads();
}

// The LDS of a sweep workgroup: the value ring and the chunk buffers, zeroed
// once per launch (inactive positions then compute zeros from zeros).
template <class V>
struct alignas(16) WfLds {
  V ring[WF_HIST * WF_RW];
  V hbuf[WF_NB * WF_CH * WF_HRW];
};
template <class V>
__device__ inline void wf_zero_lds(WfLds<V>* L) {
  constexpr int n = (int)(sizeof(WfLds<V>) / 16);
  u32x4* p = reinterpret_cast<u32x4*>(L);
  for (int i = threadIdx.x; i < n; i += WF_THREADS) p[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
}

// The last KB rows of the ring stand for the steps before a tile's first: the
// only values of the tile before that a tile reads.
template <int PAT, class V>
__device__ inline void wf_clear_history(V* ring) {
  for (int i = threadIdx.x; i < wf_kb(PAT) * WF_RW; i += WF_THREADS) ring[(WF_HIST - wf_kb(PAT)) * WF_RW + i] = V(0);
}

// What a workgroup sweeps next: a tile of a grid and the grid's strip buffer
// (0 or 1) of this sweep.
template <class V>
struct WfJob {
  WfArgs<V> a;
  unsigned tile, par;
};

// Every role of a sweep workgroup runs its own loop over the workgroup's
// tiles (values a role keeps across tiles then stay out of the other roles'
// code); next(&job) takes the next ticket, the same for all waves.
template <int PAT, int DIR, int P, class E, bool UNITD, class Next>
__device__ __forceinline__ void wf_roles(Next next, unsigned* err, WfLds<typename WfVal<E>::V>* L) {
  using V = typename WfVal<E>::V;
  WfJob<V> w;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  // this sweep's strip buffer and the one of the grid's next sweep
  auto strip = [&](unsigned other) {
    return w.a.strip + ((w.par ^ other) & 1u ? (long)w.a.t.ntx * w.a.t.nty * w.a.t.ns * wf_es(PAT) : 0l);
  };
  constexpr int CW = WF_NCW;
  if (wave < CW) {
    while (next(&w)) wf_compute<PAT, DIR, P, E, UNITD>(w.a, wf_geo(w.a, w.tile), w.tile, L->ring, L->hbuf);
  } else if (wave == CW) {
    while (next(&w)) wf_halo<PAT, DIR, V>(w.a, wf_geo(w.a, w.tile), strip(0u), L->ring, err);
  } else if (wave == CW + 1) {
    while (next(&w)) wf_load<PAT, DIR, V>(w.a, wf_geo(w.a, w.tile), L->hbuf);
  } else if (wave == CW + 2) {
    while (next(&w)) wf_store<PAT, DIR, V>(w.a, wf_geo(w.a, w.tile), L->hbuf);
  } else {
    while (next(&w))
      wf_export<PAT, DIR, V>(w.a, wf_geo(w.a, w.tile), w.tile, strip(0u), strip(1u), L->ring);
  }
}

// One sweep over one grid: persistent workgroups take tiles by ticket.
template <int PAT, int DIR, int P, class E, bool UNITD>
__global__ __launch_bounds__(WF_THREADS) void k_wavefront(WfArgs<typename WfVal<E>::V> a) {
  using V = typename WfVal<E>::V;
  __shared__ WfLds<V> L;
  SweepTickets tk(a.ctr, a.par, (unsigned)(a.t.ntx * a.t.nty));
  wf_zero_lds(&L);  // (ends with a barrier)
  tk.start();
  auto next = [&](WfJob<V>* w) {
    unsigned ticket;
    if (!tk.take(&ticket)) return false;
    w->a = a;
    // (one tile per workgroup: in the order of their index, which is a
    // dependence order too, so it needs no residence of all of them)
    const unsigned r = tk.single ? ticket : sweep_tile(ticket, a.t.sh, a.t.ntx, a.t.nty);
    w->tile = DIR > 0 ? r : tk.ntiles - 1u - r;
    w->par = tk.par;
    return true;
  };
  wf_roles<PAT, DIR, P, E, UNITD>(next, a.err, &L);
}

// One sweep over many independent grids of the same pattern and precision in
// one launch.  Ticket k names entry tmap[k] = (segment << 20) | r: the r-th
// tile of segment seg in that segment's own dependence order, so every
// tile's producers hold smaller tickets whatever the merge of the segments.
// The workgroup with the last ticket beyond the tiles (all others are done)
// readies the counter and the swept grids' buffer words for the next launch.
// (27-point FP64 keeps its deeper registers and one workgroup per CU.)
template <int PAT, int DIR, int P, class E>
__global__ __launch_bounds__(WF_THREADS, PAT == 27 && sizeof(E) == 8 ? 2 : 3) void k_wavefront_group(
    const WfArgs<typename WfVal<E>::V>* __restrict__ segs, int nseg, const unsigned* __restrict__ tmap, unsigned total,
    const int* __restrict__ live, unsigned* ctr, unsigned* err) {
  using V = typename WfVal<E>::V;
  __shared__ WfLds<V> L;
  wf_zero_lds(&L);
  bool last = false;
  auto next = [&](WfJob<V>* w) {
    for (;;) {
      const unsigned ticket = wf_take_ticket(ctr);
      if (ticket >= total) {
        last = ticket == total + gridDim.x - 1u;
        return false;
      }
      const unsigned e = __builtin_amdgcn_readfirstlane(tmap[ticket]);
      w->a = segs[e >> 20];
      if (live != nullptr && live[w->a.sys] == 0) continue;
      const unsigned r = e & 0xFFFFFu, nt = (unsigned)(w->a.t.ntx * w->a.t.nty);
      w->tile = DIR > 0 ? r : nt - 1u - r;
      w->par = __builtin_amdgcn_readfirstlane(*w->a.par);
      // (behind the ticket's barriers no wave is in a tile, and the roles start
      // with one)
      wf_clear_history<PAT>(L.ring);
      return true;
    }
  };
  wf_roles<PAT, DIR, P, E, false>(next, err, &L);
  if (last) {
    if (threadIdx.x == 0) __hip_atomic_store(&ctr[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int k = threadIdx.x; k < nseg; k += WF_THREADS)
      if (live == nullptr || live[segs[k].sys] != 0) *segs[k].par ^= 1u;
  }
}

// addout = addv + x (the correction step after an ILU(0) upper sweep)
template <class V>
__global__ __launch_bounds__(256) void k_wf_add(const V* __restrict__ addv, const V* __restrict__ x,
                                                V* __restrict__ addout, long n) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) addout[i] = addv[i] + x[i];
}

// ---------------------------------------------------------------------------
// Builds the packed schedule-ordered sweep data of one direction.  Position
// q = (tile*NS + s)*NL + lane holds the point handled there (or none); its
// element e of pack p is entry p*K + e of the list [triangle coefficients in
// canonical order, diagonal scaling] (lower triangle for dir > 0, upper for
// dir < 0); missing entries are zero.
__device__ inline long wf_point(const Grid& g, const WfTiling& tl, int pat, long q) {
  const int l = (int)(q % WF_NL);
  const long r = q / WF_NL;
  const int s = (int)(r % tl.ns);
  const int tile = (int)(r / tl.ns);
  const int X = tile / tl.nty, Y = tile % tl.nty;
  const int lx = l / WF_TY, ly = l % WF_TY;
  const int x = X * WF_TX + lx, y = Y * WF_TY + ly - tl.sh * lx;
  const int z = s - ((hp_wx(pat) - tl.sh * hp_wy(pat)) * lx + hp_wy(pat) * ly + wf_kb(pat));
  const bool v = x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
  return v ? ((long)x * g.ny + y) * g.nz + z : -1;
}

template <class E>
__device__ inline E to_e(double v);
template <>
__device__ inline double to_e<double>(double v) {
  return v;
}
template <>
__device__ inline float to_e<float>(double v) {
  return (float)v;
}

template <int PAT, class E>
__global__ __launch_bounds__(256) void k_wf_pack(Grid g, WfTiling tl, int dir, const double* __restrict__ lo,
                                                 const double* __restrict__ dg, const double* __restrict__ up,
                                                 E* __restrict__ out) {
  constexpr int C = PAT / 2, NT = PAT / 2, K = 16 / (int)sizeof(E), NPK = wf_npk(PAT, sizeof(E));
  // consecutive steps of a tile read the same column lines: keep them on one
  // XCD's L2 (contiguous block ranges per XCD)
  const long q = (long)xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (q >= tl.nsk) return;
  const long i = wf_point(g, tl, PAT, q);
  const long N = g.N();
  const long row = q / WF_NL;
  const int lane = (int)(q % WF_NL);
  // positions without a point read point 0 and store zeros: every load is
  // unconditional and all of them come before the first store, so a
  // thread's loads are in flight together
  const long ic = i >= 0 ? i : 0;
  E v[NPK * K];
#pragma unroll
  for (int m = 0; m < NPK * K; ++m) {
    double x = 0.0;
    if (m < NT) x = (dir > 0 ? lo + (long)m * N : up + (long)(C + 1 + m) * N)[ic];
    if (m == NT) x = dg[ic];
    v[m] = to_e<E>(i >= 0 ? x : 0.0);
  }
#pragma unroll
  for (int p = 0; p < NPK; ++p) {
    E* o = out + ((row * NPK + p) * WF_NL + lane) * K;
#pragma unroll
    for (int e = 0; e < K; ++e) o[e] = v[p * K + e];
  }
}

// FP16 storage: the halves of the natural FP16 matrix, and (dir > 0 call)
// the pair {row scale, diagonal scaling} per position.
template <int PAT>
__global__ __launch_bounds__(256) void k_wf_pack_h(Grid g, WfTiling tl, int dir, const __half* __restrict__ a16,
                                                   const float* __restrict__ sc, const float* __restrict__ rd,
                                                   __half* __restrict__ out, float* __restrict__ sd) {
  constexpr int C = PAT / 2, NT = PAT / 2, K = 8, NPK = wf_npk(PAT, 2);
  // consecutive steps of a tile read the same column lines: keep them on one
  // XCD's L2 (contiguous block ranges per XCD)
  const long q = (long)xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (q >= tl.nsk) return;
  const long i = wf_point(g, tl, PAT, q);
  const long N = g.N();
  const long row = q / WF_NL;
  const int lane = (int)(q % WF_NL);
  // unconditional loads (point 0 for positions without a point), all before
  // the first store
  const long ic = i >= 0 ? i : 0;
  __half v[NPK * K];
#pragma unroll
  for (int m = 0; m < NPK * K; ++m) {
    __half x = __float2half_rn(0.0f);
    if (m < NT) x = (a16 + (long)(dir > 0 ? m : C + 1 + m) * N)[ic];
    v[m] = i >= 0 ? x : __float2half_rn(0.0f);
  }
  const float s0 = sc[ic], s1 = rd[ic];
  const unsigned b0 = i >= 0 ? __float_as_uint(s0) : 0u, b1 = i >= 0 ? __float_as_uint(s1) : 0u;
  if constexpr (wf_sd_in_pack(PAT)) {
    // the scalars take the last two words: halves NPK*K-4 .. NPK*K-1
    v[NPK * K - 4] = __ushort_as_half((unsigned short)(b0 & 0xffffu));
    v[NPK * K - 3] = __ushort_as_half((unsigned short)(b0 >> 16));
    v[NPK * K - 2] = __ushort_as_half((unsigned short)(b1 & 0xffffu));
    v[NPK * K - 1] = __ushort_as_half((unsigned short)(b1 >> 16));
  }
#pragma unroll
  for (int p = 0; p < NPK; ++p) {
    __half* o = out + ((row * NPK + p) * WF_NL + lane) * K;
#pragma unroll
    for (int e = 0; e < K; ++e) o[e] = v[p * K + e];
  }
  if (!wf_sd_in_pack(PAT) && dir > 0) {
    sd[2 * q] = __uint_as_float(b0);
    sd[2 * q + 1] = __uint_as_float(b1);
  }
}

template <class E>
hipError_t launch_wf_pack(int pat, const Grid& g, const WfTiling& tl, int dir, const double* lo, const double* dg,
                          const double* up, E* out, hipStream_t st) {
  const dim3 grid((unsigned)((tl.nsk + 255) / 256)), blk(256);
  if (pat == 7)
    hipLaunchKernelGGL((k_wf_pack<7, E>), grid, blk, 0, st, g, tl, dir, lo, dg, up, out);
  else if (pat == 19)
    hipLaunchKernelGGL((k_wf_pack<19, E>), grid, blk, 0, st, g, tl, dir, lo, dg, up, out);
  else if (pat == 27)
    hipLaunchKernelGGL((k_wf_pack<27, E>), grid, blk, 0, st, g, tl, dir, lo, dg, up, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
template hipError_t launch_wf_pack<double>(int, const Grid&, const WfTiling&, int, const double*, const double*,
                                           const double*, double*, hipStream_t);
template hipError_t launch_wf_pack<float>(int, const Grid&, const WfTiling&, int, const double*, const double*,
                                          const double*, float*, hipStream_t);

hipError_t launch_wf_pack_h(int pat, const Grid& g, const WfTiling& tl, int dir, const __half* a16, const float* sc,
                            const float* rd, __half* out, float* sd, hipStream_t st) {
  const dim3 grid((unsigned)((tl.nsk + 255) / 256)), blk(256);
  if (pat == 7)
    hipLaunchKernelGGL((k_wf_pack_h<7>), grid, blk, 0, st, g, tl, dir, a16, sc, rd, out, sd);
  else if (pat == 19)
    hipLaunchKernelGGL((k_wf_pack_h<19>), grid, blk, 0, st, g, tl, dir, a16, sc, rd, out, sd);
  else if (pat == 27)
    hipLaunchKernelGGL((k_wf_pack_h<27>), grid, blk, 0, st, g, tl, dir, a16, sc, rd, out, sd);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
template <int PAT, int DIR, int P, class E, bool UNITD>
static hipError_t launch_wf_t(const WfArgs<typename WfVal<E>::V>& a, hipStream_t st) {
  const unsigned ntiles = (unsigned)(a.t.ntx * a.t.nty);
  const unsigned grid = ntiles < (unsigned)WF_MAX_GRID ? ntiles : (unsigned)WF_MAX_GRID;
  hipLaunchKernelGGL((k_wavefront<PAT, DIR, P, E, UNITD>), dim3(grid), dim3(WF_THREADS), 0, st, a);
  return hipGetLastError();
}

template <int PAT, int DIR, int P, class E>
static hipError_t launch_wfg_t(const WfArgs<typename WfVal<E>::V>* segs, int nseg, const unsigned* tmap, unsigned total,
                               unsigned grid, const int* live, unsigned* ctr, unsigned* err, hipStream_t st) {
  hipLaunchKernelGGL((k_wavefront_group<PAT, DIR, P, E>), dim3(grid), dim3(WF_THREADS), 0, st, segs, nseg, tmap, total,
                     live, ctr, err);
  return hipGetLastError();
}

// Coefficient prefetch distance (steps) per pattern and storage type: as deep
// as regs registers hold (NPK 16-byte packs per step).  A launch of one grid
// has one workgroup per CU (256 registers a lane); grouped launches have two
// (168), which hide each other's waits: 256 systems of 16..96 points per axis
// solve in 156 instead of 168 ms (FP32).
template <int PAT, class E>
constexpr int wf_prefetch(int regs = 160) {
  return wf_npk(PAT, sizeof(E)) * 4 * 16 <= regs ? 16 : (wf_npk(PAT, sizeof(E)) * 4 * 8 <= regs ? 8 : 4);
}

template <class E>
hipError_t launch_wavefront(int pat, int dir, bool unitd, bool add, const WfArgs<typename WfVal<E>::V>& a,
                            hipStream_t st) {
  using V = typename WfVal<E>::V;
  hipError_t e = hipErrorInvalidValue;
#define SMG_WF_CASE(PATV)                                                                           \
  if (pat == PATV) {                                                                                \
    constexpr int PV = wf_prefetch<PATV, E>();                                                      \
    if (dir > 0 && !unitd) e = launch_wf_t<PATV, 1, PV, E, false>(a, st);                           \
    if (dir < 0 && !unitd) e = launch_wf_t<PATV, -1, PV, E, false>(a, st);                          \
    if (dir > 0 && unitd) e = launch_wf_t<PATV, 1, PV, E, true>(a, st);                             \
  }
  SMG_WF_CASE(7)
  SMG_WF_CASE(19)
  SMG_WF_CASE(27)
#undef SMG_WF_CASE
  if (e != hipSuccess || !add) return e;
  // addout = addv + x once the sweep has finished
  const long n = a.g.N();
  hipLaunchKernelGGL((k_wf_add<V>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a.addv,
                     (const V*)a.x, a.addout, n);
  return hipGetLastError();
}

template hipError_t launch_wavefront<double>(int, int, bool, bool, const WfArgs<double>&, hipStream_t);
template hipError_t launch_wavefront<float>(int, int, bool, bool, const WfArgs<float>&, hipStream_t);
template hipError_t launch_wavefront<__half>(int, int, bool, bool, const WfArgs<float>&, hipStream_t);

// (Behind the sweeps of one grid, so that a change here does not move their code:
// FP16 27-point sweeps took 1% more at other addresses.)
template <class E>
hipError_t launch_wavefront_group(int pat, int dir, const WfArgs<typename WfVal<E>::V>* segs, int nseg,
                                  const unsigned* tmap, unsigned total, unsigned grid, const int* live, unsigned* ctr,
                                  unsigned* err, hipStream_t st) {
  if (total == 0) return hipSuccess;
  if (grid == 0 || grid > (unsigned)WF_MAX_GRID) grid = WF_MAX_GRID;
  grid = 2 * grid < total ? 2 * grid : total;
#define SMG_WFG_CASE(PATV)                                                                                       \
  if (pat == PATV && dir > 0)                                                                                    \
    return launch_wfg_t<PATV, 1, wf_prefetch<PATV, E>(112), E>(segs, nseg, tmap, total, grid, live, ctr, err, st);         \
  if (pat == PATV && dir < 0)                                                                                    \
    return launch_wfg_t<PATV, -1, wf_prefetch<PATV, E>(112), E>(segs, nseg, tmap, total, grid, live, ctr, err, st);
  SMG_WFG_CASE(7)
  SMG_WFG_CASE(19)
  SMG_WFG_CASE(27)
#undef SMG_WFG_CASE
  return hipErrorInvalidValue;
}
template hipError_t launch_wavefront_group<double>(int, int, const WfArgs<double>*, int, const unsigned*, unsigned,
                                                   unsigned, const int*, unsigned*, unsigned*, hipStream_t);
template hipError_t launch_wavefront_group<float>(int, int, const WfArgs<float>*, int, const unsigned*, unsigned,
                                                   unsigned, const int*, unsigned*, unsigned*, hipStream_t);
template hipError_t launch_wavefront_group<__half>(int, int, const WfArgs<float>*, int, const unsigned*, unsigned,
                                                   unsigned, const int*, unsigned*, unsigned*, hipStream_t);

}  // namespace smg
