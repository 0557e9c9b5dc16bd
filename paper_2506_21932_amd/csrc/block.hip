// 3x3 block systems (vector PDEs, the block operators of Sec. 4.2.3 and the
// elasticity problem of Sec. 5.1): point-block SpMV and residual, the input
// of the backward post-smoothing sweep, and the dependence-preserving
// point-block Gauss-Seidel sweep (Sec. 4.4 with 3x3 blocks).
//
// Storage: entry (r, c) of the block of offset s at A[(s*9 + r*3 + c)*N + i];
// vectors interleaved v[i*3 + c].  Per scalar row r of a block row the
// accumulation runs over neighbour blocks in canonical order and, inside a
// block, over columns c in order, with fma.
//
// The block sweep follows the scalar wavefront design (csrc/wavefront.hip):
// z-columns in sheared tiles taken by ticket in dependence order, per-column
// skew with the 3d27 hyperplane weights (4, 2, 1), one barrier per step, an
// LDS ring for neighbour values, strips of exported values between tiles, and
// waves by role (compute, halo, load, store, export).  A node has 3 values and
// needs 13 coefficient blocks and the inverse diagonal block per step (126
// numbers, 1 KB in FP64).  So a tile is 4 x 8 columns, and a compute wave holds
// 16 columns, four lanes each: lane r < 3 accumulates scalar row r (42
// numbers, in the oracle's order), the three sums meet through quad
// broadcasts, and each lane applies its row of the inverse.  A step is bound
// by the chain of 39 dependent fmas (forward: 24 of them are two or more steps
// old and summed one step early) and by the CU's own load rate (17 KB a step in
// FP32, 32 KB in FP64); the values a step needs are read from LDS in batches
// ahead of the chain.  Forward sweep before (8 x 8 tiles, a wave per scalar
// row that also did the halo loads and all stores, two barriers per step) /
// after, MI355X: 128^3 FP32 2300 / 600 us (its 1.06 GB of coefficients take
// 226 us at the 4.7 TB/s of a large copy), 64^3 1010 / 271 us; 45x52x39 FP64
// 820 / 343 us.
#include "smg_common.h"
#include "smg_group.h"
#include "smg_kernels.h"
#include "smg_sweep.h"

namespace smg {

// ------------------------------------------------------------ SpMV / residual
template <class M, bool RES>
__global__ __launch_bounds__(256) void k_bspmv(Grid g, M m, const typename M::V* __restrict__ x,
                                               const typename M::V* __restrict__ b, typename M::V* __restrict__ y,
                                               const double* gate) {
  using V = typename M::V;
  if (gate != nullptr && *gate == 0.0) return;
  const long N = g.N();
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  const int X = (int)(i / ((long)g.ny * g.nz)), Y = (int)((i / g.nz) % g.ny), Z = (int)(i % g.nz);
  // A rolled loop over the nine (dx, dy) columns of neighbours: their three
  // nodes' values and 27 coefficients are loaded together, without branches
  // (a neighbour off the grid reads the row's own node and its terms are left
  // out).  Unrolled over all 243 terms, the code itself and its branches bound
  // a small level, whose waves run it once.  Unrolled / rolled: 128^3 FP32
  // residual 449 / 379 us, 128^3 FP64 product 923 / 799 us (4.2 GB), 8^3 FP32
  // 41 / 12 us, 22x26x19 FP64 47 / 18 us.
  V acc[3] = {V(0), V(0), V(0)};
#pragma unroll 1
  for (int k = 0; k < 9; ++k) {
    const int dx = k / 3 - 1, dy = k % 3 - 1;
    const bool okxy = X + dx >= 0 && X + dx < g.nx && Y + dy >= 0 && Y + dy < g.ny;
    const long jc = okxy ? i + ((long)dx * g.ny + dy) * g.nz : i;
    V cf[27], xv[9];
    bool ok[3];
#pragma unroll
    for (int z = 0; z < 3; ++z) {
      ok[z] = okxy && Z + z - 1 >= 0 && Z + z - 1 < g.nz;
      const long j = ok[z] ? jc + z - 1 : i;
#pragma unroll
      for (int c = 0; c < 3; ++c) xv[z * 3 + c] = x[j * 3 + c];
#pragma unroll
      for (int e = 0; e < 9; ++e) cf[z * 9 + e] = m((k * 3 + z) * 9 + e, e / 3, i);
    }
#pragma unroll
    for (int z = 0; z < 3; ++z)
#pragma unroll
      for (int e = 0; e < 9; ++e) acc[e / 3] = ok[z] ? fma(cf[z * 9 + e], xv[z * 3 + e % 3], acc[e / 3]) : acc[e / 3];
  }
#pragma unroll
  for (int r = 0; r < 3; ++r) y[i * 3 + r] = RES ? b[i * 3 + r] - acc[r] : acc[r];
}

template <class M>
hipError_t launch_bspmv(const Grid& g, const M& m, const typename M::V* x, const typename M::V* b,
                        typename M::V* y, bool res, hipStream_t st) {
  const dim3 grid((unsigned)((g.N() + 255) / 256)), blk(256);
  if (res)
    hipLaunchKernelGGL((k_bspmv<M, true>), grid, blk, 0, st, g, m, x, b, y, (const double*)nullptr);
  else
    hipLaunchKernelGGL((k_bspmv<M, false>), grid, blk, 0, st, g, m, x, b, y, (const double*)nullptr);
  return hipGetLastError();
}

hipError_t launch_bspmv_res_gated(const Grid& g, const BMatD& m, const double* x, const double* b, double* y,
                                  const double* gate, hipStream_t st) {
  const dim3 grid((unsigned)((g.N() + 255) / 256)), blk(256);
  hipLaunchKernelGGL((k_bspmv<BMatD, true>), grid, blk, 0, st, g, m, x, b, y, gate);
  return hipGetLastError();
}

// h = f - sum over lower (UP = false) or upper (UP = true) neighbour blocks
// of A_ij u_j (old values): the terms a backward or forward sweep takes from
// before the sweep, in the order the sequential sweep applies them (first
// group of the row update).
template <class M, bool UP>
__global__ __launch_bounds__(256) void k_btri(Grid g, M m, const typename M::V* __restrict__ f,
                                              const typename M::V* __restrict__ u, typename M::V* __restrict__ h) {
  using V = typename M::V;
  const long N = g.N();
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  const int X = (int)(i / ((long)g.ny * g.nz)), Y = (int)((i / g.nz) % g.ny), Z = (int)(i % g.nz);
  const long nyz = (long)g.ny * g.nz;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    V t = f[i * 3 + r];
#pragma unroll
    for (int s = UP ? 14 : 0; s < (UP ? 27 : 13); ++s) {
      const int dx = pat_off(27, s, 0), dy = pat_off(27, s, 1), dz = pat_off(27, s, 2);
      if (!in_grid(g, X + dx, Y + dy, Z + dz)) continue;
      const long j = i + dx * nyz + dy * g.nz + dz;
#pragma unroll
      for (int c = 0; c < 3; ++c) t = fma(-m(s * 9 + r * 3 + c, r, i), u[j * 3 + c], t);
    }
    h[i * 3 + r] = t;
  }
}

template <class M>
hipError_t launch_blower(const Grid& g, const M& m, const typename M::V* f, const typename M::V* u,
                         typename M::V* h, hipStream_t st) {
  hipLaunchKernelGGL((k_btri<M, false>), dim3((unsigned)((g.N() + 255) / 256)), dim3(256), 0, st, g, m, f, u, h);
  return hipGetLastError();
}

template <class M>
hipError_t launch_bupper(const Grid& g, const M& m, const typename M::V* f, const typename M::V* u,
                         typename M::V* h, hipStream_t st) {
  hipLaunchKernelGGL((k_btri<M, true>), dim3((unsigned)((g.N() + 255) / 256)), dim3(256), 0, st, g, m, f, u, h);
  return hipGetLastError();
}

#define SMG_BINST(M)                                                                                           \
  template hipError_t launch_bspmv<M>(const Grid&, const M&, const M::V*, const M::V*, M::V*, bool, hipStream_t); \
  template hipError_t launch_blower<M>(const Grid&, const M&, const M::V*, const M::V*, M::V*, hipStream_t); \
  template hipError_t launch_bupper<M>(const Grid&, const M&, const M::V*, const M::V*, M::V*, hipStream_t);
SMG_BINST(BMatD)
SMG_BINST(BMatF)
SMG_BINST(BMatH)
#undef SMG_BINST

// ------------------------------------------------------------ block sweep
constexpr int BW_TX = 4, BW_TY = 8, BW_NL = BW_TX * BW_TY;  // columns per tile
constexpr int BW_HIST = 16;                  // LDS ring rows (steps)
constexpr int BW_CH = 16;                    // steps per chunk of right-hand side / results
constexpr int BW_NB = 3;                     // chunk buffers: filled, computed, drained
constexpr int BW_NH = 12 + 2 * BW_TX;        // halo slots (nodes) around a tile
constexpr int BW_NCW = BW_NL / 16;           // compute waves, 16 columns each
constexpr int BW_THREADS = 64 * (BW_NCW + 4);  // ... and a halo, a load, a store and an export wave
constexpr int BW_RW = (BW_NL + BW_NH) * 4;   // ring row length (a node takes 4 entries)
constexpr int BW_HRW = BW_NL * 4 + 1;        // chunk buffer row length (padded)
constexpr int BW_GRP = BW_NL / 4;            // groups of 4 columns; a group's run of 16 steps is 3 x 64 values
constexpr int BW_LPS = 2;                    // runs moved per step (the last are done before step 14)
constexpr int BW_ES = 3 * (BW_TY + 2 * BW_TX);  // strip entries per step
constexpr int BW_PH = 4;                     // halo prefetch distance (steps)
constexpr int BW_AHEAD = BW_PH + 2;          // steps a stalled tile falls back behind its producer
constexpr int BW_WX = 4, BW_WY = 2, BW_KB = 7;  // 3d27 hyperplane weights, largest lower step distance
static_assert(3 * BW_NH <= 64 && BW_ES <= 64 && 3 * BW_GRP <= BW_LPS * (BW_CH - 2), "one wave per role");

static void bw_tile(const Grid& g, WfTiling* t, int tx) {
  t->sh = g.ny <= BW_TY ? 0 : 1;
  t->ntx = (g.nx + tx - 1) / tx;
  t->nty = (g.ny + t->sh * (tx - 1) + BW_TY - 1) / BW_TY;
  t->ns = g.nz + (BW_WX - t->sh * BW_WY) * (tx - 1) + BW_WY * (BW_TY - 1) + 2 * BW_KB;
  t->nsk = (long)t->ntx * t->nty * t->ns * tx * BW_TY;
}
void bwf_tiling(const Grid& g, WfTiling* t) { bw_tile(g, t, BW_TX); }
long bwf_reserve(const Grid& g) {
  WfTiling t;
  bw_tile(g, &t, 8);
  return t.nsk;
}
long bwf_strip_elems(const WfTiling& t) { return (long)t.ntx * t.nty * t.ns * BW_ES; }

// Sweep data per node and scalar row r: the row's 13 triangle blocks (3
// entries each, canonical order) then row r of the inverse diagonal block.
// FP64: 42 doubles = 21 packs; FP32: 42 floats in 11 packs; FP16: 39 halves
// (bytes 0..77), the FP32 row scale (byte 80) and the FP32 inverse row
// (bytes 84..95) = 6 packs.  Layout [tile][step][pack][column * 3 + r].
__host__ __device__ constexpr int bwf_npr(int ebytes) { return ebytes == 8 ? 21 : (ebytes == 4 ? 11 : 6); }
int bwf_pack_count(int ebytes) { return 3 * bwf_npr(ebytes); }

// Term m of the triangle (canonical order): neighbour column (forward frame)
// and step distance.
__host__ __device__ constexpr int bw_off(int dir, int m, int axis) { return pat_off(27, dir > 0 ? m : 14 + m, axis); }
__host__ __device__ constexpr int bw_back(int dir, int m) {
  return dir * (BW_WX * bw_off(dir, m, 0) + BW_WY * bw_off(dir, m, 1) + bw_off(dir, m, 2));
}
// leading terms whose values are at least two steps old
__host__ __device__ constexpr int bw_prefix(int dir) {
  int n = 0;
  while (n < 13 && bw_back(dir, n) <= -2) ++n;
  return n;
}

// Halo nodes, export entries: as in the scalar sweep (forward frame: the
// column x-1 with y in [-2, TY+2), the row y = -1, a second row; the TY
// columns lx = TX-1, the TX columns ly = TY-1, the TX columns of the second
// row), three values each.
__host__ __device__ constexpr int bw_halo_slot(int dir, int qx, int qy) {
  const int fx = dir > 0 ? qx : BW_TX - 1 - qx, fy = dir > 0 ? qy : BW_TY - 1 - qy;
  return fx < 0 ? fy + 2 : (fy == -1 ? 12 + fx : 12 + BW_TX + fx);
}
__device__ inline void bw_halo_pos(int sh, int n, int* fx, int* fy) {
  *fx = n < 12 ? -1 : (n < 12 + BW_TX ? n - 12 : n - 12 - BW_TX);
  *fy = n < 12 ? n - 2 : (n < 12 + BW_TX ? -1 : (sh ? -2 : BW_TY));
}
// Is forward-frame node (fx, fy) a lower neighbour column of some lane?
__device__ inline bool bw_halo_used(int sh, int fx, int fy) {
  for (int c = 0; c < 4; ++c) {
    const int cx = c == 3 ? 0 : -1, cy = c == 3 ? -1 : c - 1;
    const int lx = fx - cx, ly = fy - cy - sh * cx;
    if (lx >= 0 && lx < BW_TX && ly >= 0 && ly < BW_TY) return true;
  }
  return false;
}
__device__ inline int bw_export_lane(int dir, int sh, int e) {
  int lx = e < BW_TY ? BW_TX - 1 : (e - BW_TY) % BW_TX;
  int ly = e < BW_TY ? e : (e < BW_TY + BW_TX ? BW_TY - 1 : (sh ? BW_TY - 2 : 0));
  if (dir < 0) {
    lx = BW_TX - 1 - lx;
    ly = BW_TY - 1 - ly;
  }
  return lx * BW_TY + ly;
}

// entry e (0..41) of a row's sweep data held in packs p[]: e < 39 are the
// triangle coefficients (block e / 3, column e % 3), e = 39 + c the inverse
// row's column c
template <class E>
__device__ inline typename WfVal<E>::V bw_row(const u32x4* p, int e);
template <>
__device__ inline double bw_row<double>(const u32x4* p, int e) {
  const u32x4 w = p[e / 2];
  return e % 2 == 0 ? __builtin_bit_cast(double, u32x2{w.x, w.y}) : __builtin_bit_cast(double, u32x2{w.z, w.w});
}
template <>
__device__ inline float bw_row<float>(const u32x4* p, int e) {
  return __uint_as_float(p[e / 4][e % 4]);
}
template <>
__device__ inline float bw_row<__half>(const u32x4* p, int e) {
  if (e >= 39) return __uint_as_float(p[(84 + 4 * (e - 39)) / 16][((84 + 4 * (e - 39)) % 16) / 4]);
  // row scale (byte 80) times the half, rounded once
  const unsigned w = p[e / 8][(e % 8) / 2];
  const float sc = __uint_as_float(p[5][0]);
  return e % 2 == 0 ? half_times<0>(w, sc) : half_times<1>(w, sc);
}

// v of lane 4 * (lane / 4) + R (quad broadcast)
template <int R>
__device__ inline float bw_quad(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), R * 0x55, 0xf, 0xf, true));
}
template <int R>
__device__ inline double bw_quad(double v) {
  const u32x2 w = __builtin_bit_cast(u32x2, v);
  return __builtin_bit_cast(
      double, u32x2{(unsigned)__builtin_amdgcn_mov_dpp((int)w.x, R * 0x55, 0xf, 0xf, true),
                    (unsigned)__builtin_amdgcn_mov_dpp((int)w.y, R * 0x55, 0xf, 0xf, true)});
}

struct BwGeo {
  int X, Y, sh, NS, nsteps, p0;
  unsigned vbytes;  // bytes of the vector buffers (planes p0 .. p1-1)
  long vb;          // element offset of plane p0
  bool full;        // every column of the tile lies in the grid
};
template <class V>
__device__ inline BwGeo bw_geo(const WfArgs<V>& a, unsigned tile) {
  BwGeo q;
  q.X = (int)(tile / (unsigned)a.t.nty);
  q.Y = (int)(tile % (unsigned)a.t.nty);
  q.sh = a.t.sh;
  q.NS = a.t.ns;
  q.nsteps = (q.NS + BW_CH - 1) / BW_CH * BW_CH;
  q.p0 = q.X * BW_TX > 0 ? q.X * BW_TX - 1 : 0;
  const int p1 = q.X * BW_TX + BW_TX + 1 < a.g.nx ? q.X * BW_TX + BW_TX + 1 : a.g.nx;
  const long pl = 3l * a.g.ny * a.g.nz;
  q.vbytes = (unsigned)((p1 - q.p0) * pl * (long)sizeof(V));
  q.vb = q.p0 * pl;
  const int y0 = q.Y * BW_TY;
  q.full = q.X * BW_TX + BW_TX <= a.g.nx && y0 - q.sh * (BW_TX - 1) >= 0 && y0 + BW_TY <= a.g.ny;
  return q;
}
template <int DIR>
__device__ inline int bw_step(int NS, int k) {
  return DIR > 0 ? k : NS - 1 - k;
}

// ---- compute role (the first two waves): lane 4 * column + r computes scalar
// row r of its column's node (r = 3 idles); a node's three row sums meet
// through quad broadcasts
template <int DIR, int P, class E>
__device__ __forceinline__ void bw_compute(const WfArgs<typename WfVal<E>::V>& a, const BwGeo& q, unsigned tile,
                                           typename WfVal<E>::V* ring, typename WfVal<E>::V* hbuf) {
  using V = typename WfVal<E>::V;
  constexpr int NPR = bwf_npr(sizeof(E)), K = 16 / (int)sizeof(E);
  constexpr int NPRE = bw_prefix(DIR), PPRE = 3 * NPRE / K;  // prefix terms, and the packs they fill
  constexpr int BATCH = sizeof(V) == 8 ? 4 : 13;  // nodes whose values are read ahead
  constexpr unsigned PACKB = 3 * BW_NL * 16u;
  static_assert(BW_HIST % P == 0 && BW_HIST > BW_KB + 1 && 3 * NPRE % K == 0, "prefetch");
  const int col = threadIdx.x / 4, r = threadIdx.x % 4;
  const int lx = col / BW_TY, ly = col % BW_TY;
  const int NS = q.NS;
  int nidx[4];  // ring index of each neighbour column's node
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int cx = c == 3 ? 0 : -DIR, cy = c == 3 ? -DIR : DIR * (c - 1);
    const int qx = lx + cx, qy = ly + cy + q.sh * cx;
    const bool in = qx >= 0 && qx < BW_TX && qy >= 0 && qy < BW_TY;
    nidx[c] = 4 * (in ? qx * BW_TY + qy : BW_NL + bw_halo_slot(DIR, qx, qy));
  }
  const unsigned tbytes = (unsigned)NS * NPR * PACKB;
  const auto rp = wf_rsrc((const char*)a.pk + (size_t)tile * tbytes, tbytes);
  const int skew = (BW_WX - q.sh * BW_WY) * lx + BW_WY * ly + BW_KB;
  const int xt = q.X * BW_TX + lx, yt = q.Y * BW_TY + ly - q.sh * lx;
  const unsigned zlim = xt < a.g.nx && yt >= 0 && yt < a.g.ny ? (unsigned)a.g.nz : 0u;
  const unsigned lo = r < 3 ? (unsigned)(col * 3 + r) * 16u : WF_OOB;
  auto is_point = [&](int k) { return (unsigned)(bw_step<DIR>(NS, k) - skew) < zlim; };
  // packs of step k into slot j (positions without a point read as zero
  // without a memory access)
  u32x4 cf[P][NPR];
  struct Po {
    unsigned so, vo;
  };
  auto pack_off = [&](int k) {
    const int s = bw_step<DIR>(NS, k);
    return Po{s >= 0 && s < NS ? (unsigned)s * (NPR * PACKB) : WF_OOB, is_point(k) ? lo : WF_OOB};
  };
  auto pack_load = [&](const Po& o, int j, int p) {
    cf[j][p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, o.vo, o.so + p * PACKB, 0));
  };
#pragma unroll
  for (int j = 0; j < P; ++j) {
    // (step 0 has no points: its prefix is skipped, so slot 0 starts with the
    // prefix packs of step P)
    const Po o = pack_off(j), on = pack_off(j + P);
#pragma unroll
    for (int p = 0; p < NPR; ++p) pack_load(j == 0 && p < PPRE ? on : o, j, p);
  }
  const int me = col * 4 + r;
  V own = V(0), tp;
  __syncthreads();  // prologue: the first chunk is in LDS
  tp = hbuf[me];

  for (int k0 = 0; k0 < q.nsteps; k0 += BW_HIST) {
    V* hb = hbuf + ((k0 / BW_CH) % BW_NB) * (BW_CH * BW_HRW) + me;
    const V* hbn = hbuf + ((k0 / BW_CH + 1) % BW_NB) * (BW_CH * BW_HRW) + me;
#pragma unroll
    for (int j = 0; j < BW_HIST; ++j) {
      const int jp = j % P, jn = (j + 1) % P, k = k0 + j;
      V u[13][3];
      // the values of terms m0 .. m0 + BATCH - 1 of a step; all reads are
      // issued before the first use
      auto values = [&](int m0, int m1, int step) {
#pragma unroll
        for (int m = m0; m < m0 + BATCH && m < m1; ++m) {
          if (bw_off(DIR, m, 0) == 0 && bw_off(DIR, m, 1) == 0) {
            u[m][0] = bw_quad<0>(own);
            u[m][1] = bw_quad<1>(own);
            u[m][2] = bw_quad<2>(own);
          } else {
            const int c = bw_off(DIR, m, 0) != 0 ? DIR * bw_off(DIR, m, 1) + 1 : 3;
            const V* n = ring + ((step + bw_back(DIR, m) + BW_HIST) % BW_HIST) * BW_RW + nidx[c];
#pragma unroll
            for (int i = 0; i < 3; ++i) u[m][i] = n[i];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      // t -= A_m u_m with the packs of slot
      auto term = [&](V t, int m, int slot) {
#pragma unroll
        for (int i = 0; i < 3; ++i) t = fma(-bw_row<E>(cf[slot], 3 * m + i), u[m][i], t);
        return t;
      };
      V t = tp;
      values(NPRE, 13, j);
#pragma unroll
      for (int m = NPRE; m < 13; ++m) {
        if ((m - NPRE) % BATCH == 0 && m + BATCH < 13) values(m + BATCH, 13, j);
        t = term(t, m, jp);
      }
      // row r of the inverse diagonal block times the node's three sums
      const V t0 = bw_quad<0>(t), t1 = bw_quad<1>(t), t2 = bw_quad<2>(t);
      const V xv = fma(bw_row<E>(cf[jp], 41), t2, fma(bw_row<E>(cf[jp], 40), t1, bw_row<E>(cf[jp], 39) * t0));
      own = is_point(k) ? xv : V(0);
      // (the last FP32 pack's unused words stay live until here, so that no
      // temporary waits for a load in flight)
      if constexpr (sizeof(E) == 4) asm volatile("" : : "v"(cf[jp][NPR - 1]));
      ring[j * BW_RW + me] = own;
      hb[j * BW_HRW] = own;
      __builtin_amdgcn_sched_barrier(0);
      // refill the packs used for the last time, then sum the next step's
      // prefix (its values are in the ring already)
      const Po po = pack_off(k + P), pn = pack_off(k + 1 + P);
#pragma unroll
      for (int p = PPRE; p < NPR; ++p) pack_load(po, jp, p);
      tp = j + 1 < BW_HIST ? hb[(j + 1) * BW_HRW] : hbn[0];
      if (NPRE > 0) values(0, NPRE, j + 1);
#pragma unroll
      for (int m = 0; m < NPRE; ++m) {
        if (m % BATCH == 0 && m + BATCH < NPRE) values(m + BATCH, NPRE, j + 1);
        tp = term(tp, m, jn);
#pragma unroll
        for (int p = 3 * m / K; p < 3 * (m + 1) / K; ++p) {
          __builtin_amdgcn_sched_barrier(0);
          pack_load(pn, jn, p);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
    }
  }
  __syncthreads();  // tail: the last chunk is drained and the last step exported
  __syncthreads();
}

// ---- halo role: lane 3 n + c brings component c of halo node n from the
// producing tile's strip into the ring (see the scalar sweep)
template <int DIR, class V>
__device__ __forceinline__ void bw_halo(const WfArgs<V>& a, const BwGeo& q, const V* strip, V* ring, unsigned* err) {
  using B = VBits<V>;
  constexpr int PH = BW_PH;
  static_assert(BW_CH % PH == 0, "halo prefetch distance");
  const int t = threadIdx.x - 64 * BW_NCW;
  const int NS = q.NS;
  int fx = 0, fy = 0;
  bool role = false;
  if (t < 3 * BW_NH) {
    bw_halo_pos(q.sh, t / 3, &fx, &fy);
    role = bw_halo_used(q.sh, fx, fy);
  }
  const int ax = fx < 0 ? 1 : 0;
  const int fyt = fy + (ax ? BW_TX * q.sh : 0) + 2 * BW_TY;  // >= 0
  const int dyf = fyt / BW_TY - 2, lyf = fyt % BW_TY, lxf = ax ? BW_TX - 1 : fx;
  const int PX = q.X - DIR * ax, PY = q.Y + DIR * dyf;
  const bool have = role && PX >= 0 && PX < a.t.ntx && PY >= 0 && PY < a.t.nty;
  const int dk = DIR * (BW_WX * BW_TX * ax - BW_WY * BW_TY * dyf);
  const int e = lxf == BW_TX - 1 ? lyf : (lyf == BW_TY - 1 ? BW_TY + lxf : BW_TY + BW_TX + lxf);
  const V* hp = have ? strip + (((long)PX * a.t.nty + PY) * NS) * BW_ES + 3 * e + t % 3 : strip;
  const int es = have ? BW_ES : 0;
  const int slot = 4 * (BW_NL + t / 3) + t % 3;
  auto valid = [&](int k) {
    const int s = bw_step<DIR>(NS, k), sp = s + dk;
    return have && s >= 0 && s < NS && sp >= 0 && sp < NS;
  };
  auto fetch = [&](int k) {
    int sp = bw_step<DIR>(NS, k) + dk;
    sp = sp < 0 ? 0 : (sp >= NS ? NS - 1 : sp);
    return wf_coherent_load(hp + (long)sp * es);
  };
  V hb[PH];
  auto put = [&](int k, int j) {
    const bool ok = valid(k);
    if (__builtin_amdgcn_ballot_w64(ok && B::bits(hb[j]) == B::sent) != 0) {
      unsigned spins = 0;
      for (;;) {
        const V far = fetch(k + BW_AHEAD);
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
    if (role) ring[(k % BW_HIST) * BW_RW + slot] = ok ? hb[j] : V(0);
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

// ---- column runs (load and store roles).  A chunk's 16 steps of a column are
// 48 consecutive values; run 3 g + i moves values 64 i .. 64 i + 63 of the
// four columns of group g (lx = g / 2, ly = 4 (g % 2) ..).
template <int DIR, class V>
struct BwRuns {
  int cq[3], zo[3], lds[3];  // column in the group, point in the column's run, LDS index
  unsigned vin[3];           // inner chunks: lane part of the byte offset
  int off[3];                // value in the column's run
  __device__ void init(const WfArgs<V>& a, int lane) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int e = 64 * i + lane;
      cq[i] = e / 48;
      off[i] = e % 48;
      zo[i] = off[i] / 3;
      lds[i] = (DIR > 0 ? zo[i] : BW_CH - 1 - zo[i]) * BW_HRW + 4 * cq[i] + off[i] % 3;
      vin[i] = (unsigned)(cq[i] * (a.g.nz - BW_WY) * 3 + off[i]) * (unsigned)sizeof(V);
    }
  }
  // lowest step of chunk c
  __device__ static int low(const BwGeo& q, int c) {
    return DIR > 0 ? c * BW_CH : q.NS - BW_CH - c * BW_CH;
  }
  // is every position of chunk c a point?
  __device__ static bool inner(const WfArgs<V>& a, const BwGeo& q, int c) {
    const int lo = low(q, c), sx = BW_WX - q.sh * BW_WY;
    return q.full && lo >= BW_KB + sx * (BW_TX - 1) + BW_WY * (BW_TY - 1) && lo + BW_CH - 1 - BW_KB < a.g.nz;
  }
  // offsets (vector and scalar part) of run 3 g + i of chunk c
  __device__ void offset(const WfArgs<V>& a, const BwGeo& q, int c, bool in, int g, int i, unsigned* vo,
                         unsigned* so) const {
    const int lx = g / 2, y0 = 4 * (g % 2), sx = BW_WX - q.sh * BW_WY;
    const int lo = wf_keep_s(low(q, c)) - BW_KB - sx * lx - BW_WY * y0;  // z of the group's first column
    const int row = (q.X * BW_TX - q.p0 + lx) * a.g.ny + q.Y * BW_TY + y0 - q.sh * lx;
    if (in) {
      *vo = vin[i];
      *so = (unsigned)((row * a.g.nz + lo) * 3) * (unsigned)sizeof(V);
    } else {
      const int y = q.Y * BW_TY + y0 + cq[i] - q.sh * lx, z = lo - BW_WY * cq[i] + zo[i];
      const bool ok = q.X * BW_TX + lx < a.g.nx && (unsigned)y < (unsigned)a.g.ny && (unsigned)z < (unsigned)a.g.nz;
      const int e = ((row + cq[i]) * a.g.nz + lo - BW_WY * cq[i]) * 3 + off[i];
      *vo = ok ? (unsigned)e * (unsigned)sizeof(V) : WF_OOB;
      *so = 0u;
    }
  }
};

// ---- load role: right-hand side, two chunks ahead
template <int DIR, class V>
__device__ __forceinline__ void bw_load(const WfArgs<V>& a, const BwGeo& q, V* hbuf) {
  constexpr int NR = 3 * BW_GRP;
  BwRuns<DIR, V> R;
  R.init(a, threadIdx.x - 64 * (BW_NCW + 1));
  const auto rh = wf_rsrc(a.h + q.vb, q.vbytes);
  V reg[NR];
  // per step two runs: registers to the chunk buffer hb, then the runs of chunk c
  auto advance = [&](V* hb, int c, bool put, bool sync) {
    const bool in = R.inner(a, q, c);
#pragma unroll
    for (int j = 0; j < BW_CH; ++j) {
#pragma unroll
      for (int i = BW_LPS * j; i < BW_LPS * (j + 1); ++i) {
        if (i >= NR) break;
        if (put) hb[R.lds[i % 3] + 16 * (i / 3)] = reg[i];
        unsigned vo, so;
        R.offset(a, q, c, in, i / 3, i % 3, &vo, &so);
        reg[i] = bld<V, 0>(rh, vo, so);
      }
      if (sync)
        __syncthreads();
      else
        __builtin_amdgcn_sched_barrier(0);
    }
  };
  // prologue: chunk 0 into buffer 0, chunk 1 into the registers
  advance(hbuf, 0, false, false);
  advance(hbuf, 1, true, false);
  __syncthreads();
  for (int c = 0; c < q.nsteps / BW_CH; ++c) advance(hbuf + ((c + 1) % BW_NB) * (BW_CH * BW_HRW), c + 2, true, true);
  __syncthreads();
  __syncthreads();
}

// ---- store role: results, one chunk behind
template <int DIR, class V>
__device__ __forceinline__ void bw_store(const WfArgs<V>& a, const BwGeo& q, const V* hbuf) {
  constexpr int NR = 3 * BW_GRP;
  BwRuns<DIR, V> R;
  R.init(a, threadIdx.x - 64 * (BW_NCW + 2));
  const auto rx = wf_rsrc(a.x + q.vb, q.vbytes);
  auto chunk = [&](int c, bool sync) {
    const V* hb = hbuf + (c % BW_NB) * (BW_CH * BW_HRW);
    const bool in = R.inner(a, q, c);
#pragma unroll
    for (int j = 0; j < BW_CH; ++j) {
#pragma unroll
      for (int i = BW_LPS * j; i < BW_LPS * (j + 1); ++i) {
        if (i >= NR) break;
        unsigned vo, so;
        R.offset(a, q, c, in, i / 3, i % 3, &vo, &so);
        bst<0>(hb[R.lds[i % 3] + 16 * (i / 3)], rx, vo, so);
      }
      if (sync) __syncthreads();
    }
  };
  __syncthreads();  // prologue
#pragma unroll 1
  for (int j = 0; j < BW_CH; ++j) __syncthreads();
  for (int c = 1; c < q.nsteps / BW_CH; ++c) chunk(c - 1, true);
  __syncthreads();
  chunk(q.nsteps / BW_CH - 1, false);
  __syncthreads();
}

// ---- export role: one step after a node is computed its values go to this
// sweep's strip buffer, and the other buffer's entries get the sentinel
template <int DIR, class V>
__device__ __forceinline__ void bw_export(const WfArgs<V>& a, const BwGeo& q, unsigned tile, V* strip, V* other,
                                          const V* ring) {
  using B = VBits<V>;
  const int e = threadIdx.x - 64 * (BW_NCW + 3);
  const bool role = e < BW_ES;
  const int el = role ? 4 * bw_export_lane(DIR, q.sh, e / 3) + e % 3 : 0;
  const long base = (long)tile * q.NS * BW_ES + e;
  auto step = [&](int k) {
    if (role && k >= 0 && k < q.NS) {
      const long o = base + (long)bw_step<DIR>(q.NS, k) * BW_ES;
      wf_coherent_store(strip + o, ring[(k % BW_HIST) * BW_RW + el]);
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

template <class V>
struct alignas(16) BwLds {
  V ring[BW_HIST * BW_RW];
  V hbuf[BW_NB * BW_CH * BW_HRW];
};

template <int DIR, int P, class E>
__global__ __launch_bounds__(BW_THREADS) void k_bwavefront(WfArgs<typename WfVal<E>::V> a) {
  using V = typename WfVal<E>::V;
  __shared__ BwLds<V> L;
  SweepTickets tk(a.ctr, a.par, (unsigned)(a.t.ntx * a.t.nty));
  // values of positions without a point stay finite
  for (int i = threadIdx.x; i < (int)(sizeof(L) / 16); i += BW_THREADS)
    reinterpret_cast<u32x4*>(&L)[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  tk.start();
  const long half = (long)a.t.ntx * a.t.nty * a.t.ns * BW_ES;
  V* const strip = a.strip + (tk.par & 1u ? half : 0l);
  V* const other = a.strip + (tk.par & 1u ? 0l : half);
  unsigned ticket;
  auto take = [&] {
    if (!tk.take(&ticket)) return false;
    if (!tk.single) ticket = sweep_tile(ticket, a.t.sh, a.t.ntx, a.t.nty);
    return true;
  };
  auto tile = [&] { return DIR > 0 ? ticket : tk.ntiles - 1u - ticket; };
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  if (wave < BW_NCW) {
    while (take()) bw_compute<DIR, P, E>(a, bw_geo(a, tile()), tile(), L.ring, L.hbuf);
  } else if (wave == BW_NCW) {
    while (take()) bw_halo<DIR, V>(a, bw_geo(a, tile()), strip, L.ring, a.err);
  } else if (wave == BW_NCW + 1) {
    while (take()) bw_load<DIR, V>(a, bw_geo(a, tile()), L.hbuf);
  } else if (wave == BW_NCW + 2) {
    while (take()) bw_store<DIR, V>(a, bw_geo(a, tile()), L.hbuf);
  } else {
    while (take()) bw_export<DIR, V>(a, bw_geo(a, tile()), tile(), strip, other, L.ring);
  }
}

template <class E>
hipError_t launch_bwavefront(int dir, const WfArgs<typename WfVal<E>::V>& a, hipStream_t st) {
  const unsigned ntiles = (unsigned)(a.t.ntx * a.t.nty);
  const unsigned grid = ntiles < (unsigned)WF_MAX_GRID ? ntiles : (unsigned)WF_MAX_GRID;
  // steps of row data fetched ahead, as the registers allow (the forward
  // sweep's prefix holds 24 more values)
  constexpr int PF = sizeof(E) == 2 ? 4 : 2, PB = sizeof(E) == 8 ? 2 : 4;
  if (dir > 0)
    hipLaunchKernelGGL((k_bwavefront<1, PF, E>), dim3(grid), dim3(BW_THREADS), 0, st, a);
  else
    hipLaunchKernelGGL((k_bwavefront<-1, PB, E>), dim3(grid), dim3(BW_THREADS), 0, st, a);
  return hipGetLastError();
}
template hipError_t launch_bwavefront<double>(int, const WfArgs<double>&, hipStream_t);
template hipError_t launch_bwavefront<float>(int, const WfArgs<float>&, hipStream_t);
template hipError_t launch_bwavefront<__half>(int, const WfArgs<float>&, hipStream_t);

// ------------------------------------------------------------ packing (setup)
__device__ inline long bwf_point(const Grid& g, const WfTiling& tl, long q) {
  const int l = (int)(q % BW_NL);
  const long r = q / BW_NL;
  const int s = (int)(r % tl.ns);
  const int tile = (int)(r / tl.ns);
  const int X = tile / tl.nty, Y = tile % tl.nty;
  const int lx = l / BW_TY, ly = l % BW_TY;
  const int x = X * BW_TX + lx, y = Y * BW_TY + ly - tl.sh * lx;
  const int z = s - ((BW_WX - tl.sh * BW_WY) * lx + BW_WY * ly + BW_KB);
  const bool v = x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
  return v ? ((long)x * g.ny + y) * g.nz + z : -1;
}

// FP64 / FP32: row r of position q: entries 3m + c = block (dir > 0 ? m :
// 14 + m) entry (r, c), m < 13; entries 39 + c = inverse diagonal entry
// (r, c); padding zero.
template <class E>
__global__ __launch_bounds__(256) void k_bwf_pack(Grid g, WfTiling tl, int dir, const double* __restrict__ A,
                                                  const double* __restrict__ Dinv, E* __restrict__ out) {
  constexpr int K = 16 / (int)sizeof(E), NPR = bwf_npr(sizeof(E));
  // consecutive steps of a tile read the same column lines: keep them on one
  // XCD's L2 (contiguous block ranges per XCD)
  // (a thread per row, so that a step's packs are stored contiguously: 45x52x39
  // FP64 231 -> 128 us, 128^3 FP32 3.8 -> 3.2 ms)
  const long t = (long)xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  const long q = t / 3;
  const int r = (int)(t % 3);
  if (q >= tl.nsk) return;
  const long i = bwf_point(g, tl, q);
  const long N = g.N();
  const long pos = q / BW_NL;
  const int lane = (int)(q % BW_NL);
  for (int p = 0; p < NPR; ++p) {
    E* o = out + ((pos * NPR + p) * (3 * BW_NL) + 3 * lane + r) * K;
    for (int e = 0; e < K; ++e) {
      const int v = p * K + e;
      double x = 0.0;
      if (i >= 0 && v < 39)
        x = A[((long)(dir > 0 ? v / 3 : 14 + v / 3) * 9 + r * 3 + v % 3) * N + i];
      else if (i >= 0 && v < 42)
        x = Dinv[(long)(r * 3 + v - 39) * N + i];
      o[e] = (E)x;
    }
  }
}

// FP16: row r of position q: the 39 halves of the row's triangle entries
// (bytes 0..77), the FP32 row scale (bytes 80..83), the FP32 inverse row
// (bytes 84..95).
__global__ __launch_bounds__(256) void k_bwf_pack_h(Grid g, WfTiling tl, int dir, const __half* __restrict__ a16,
                                                    const float* __restrict__ sc, const float* __restrict__ rd,
                                                    unsigned char* __restrict__ out) {
  constexpr int NPR = bwf_npr(2);
  // consecutive steps of a tile read the same column lines: keep them on one
  // XCD's L2 (contiguous block ranges per XCD)
  const long q = (long)xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (q >= tl.nsk) return;
  const long i = bwf_point(g, tl, q);
  const long N = g.N();
  const long pos = q / BW_NL;
  const int lane = (int)(q % BW_NL);
  for (int r = 0; r < 3; ++r) {
    unsigned char bytes[16 * NPR];
    for (int b = 0; b < 16 * NPR; ++b) bytes[b] = 0;
    for (int v = 0; v < 39; ++v) {
      const __half h = i >= 0 ? a16[((long)(dir > 0 ? v / 3 : 14 + v / 3) * 9 + r * 3 + v % 3) * N + i]
                              : __float2half_rn(0.0f);
      const unsigned short u = __half_as_ushort(h);
      bytes[2 * v] = (unsigned char)(u & 0xff);
      bytes[2 * v + 1] = (unsigned char)(u >> 8);
    }
    const unsigned us = __float_as_uint(i >= 0 ? sc[(long)r * N + i] : 0.0f);
    for (int b = 0; b < 4; ++b) bytes[80 + b] = (unsigned char)(us >> (8 * b));
    for (int c = 0; c < 3; ++c) {
      const unsigned u = __float_as_uint(i >= 0 ? rd[(long)(r * 3 + c) * N + i] : 0.0f);
      for (int b = 0; b < 4; ++b) bytes[84 + 4 * c + b] = (unsigned char)(u >> (8 * b));
    }
    for (int p = 0; p < NPR; ++p) {
      unsigned char* o = out + ((pos * NPR + p) * (3 * BW_NL) + 3 * lane + r) * 16;
      for (int b = 0; b < 16; ++b) o[b] = bytes[16 * p + b];
    }
  }
}

template <class E>
hipError_t launch_bwf_pack(const Grid& g, const WfTiling& tl, int dir, const double* A, const double* Dinv, E* out,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_bwf_pack<E>), dim3((unsigned)((3 * tl.nsk + 255) / 256)), dim3(256), 0, st, g, tl, dir, A, Dinv,
                     out);
  return hipGetLastError();
}
template hipError_t launch_bwf_pack<double>(const Grid&, const WfTiling&, int, const double*, const double*, double*,
                                            hipStream_t);
template hipError_t launch_bwf_pack<float>(const Grid&, const WfTiling&, int, const double*, const double*, float*,
                                           hipStream_t);

hipError_t launch_bwf_pack_h(const Grid& g, const WfTiling& tl, int dir, const __half* a16, const float* sc,
                             const float* rd, void* out, hipStream_t st) {
  hipLaunchKernelGGL(k_bwf_pack_h, dim3((unsigned)((tl.nsk + 255) / 256)), dim3(256), 0, st, g, tl, dir, a16, sc,
                     rd, (unsigned char*)out);
  return hipGetLastError();
}

}  // namespace smg
