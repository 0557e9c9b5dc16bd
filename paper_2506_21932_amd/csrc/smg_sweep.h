// Pieces shared by the tiled sweeps (wavefront.hip, block.hip): buffer and
// device-coherent accesses, tickets.
#pragma once
#include "smg_common.h"

namespace smg {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned WF_OOB = 0x80000000u;  // buffer offset outside every range
constexpr int WF_SC1 = 16;                // cache policy of device-coherent accesses
constexpr unsigned WF_SPIN_LIMIT = 1u << 21;

// ---- buffer access helpers -------------------------------------------------
__device__ inline __amdgpu_buffer_rsrc_t wf_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
template <class V, int CP>
__device__ inline V bld(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff = 0u) {
  if constexpr (sizeof(V) == 8)
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, CP));
  else
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, CP));
}
template <int CP, class V>
__device__ inline void bst(V v, __amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff = 0u) {
  if constexpr (sizeof(V) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, soff, CP);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, soff, CP);
}

template <class V>
__device__ inline V wf_coherent_load(const V* p) {
  using U = typename VBits<V>::U;
  return VBits<V>::val(__hip_atomic_load(reinterpret_cast<const U*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
template <class V>
__device__ inline void wf_coherent_store(V* p, V v) {
  using U = typename VBits<V>::U;
  __hip_atomic_store(reinterpret_cast<U*>(p), VBits<V>::bits(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keeps the compiler from moving the computation of v across memory operations.
__device__ inline int wf_keep(int v) {
  asm volatile("" : "+v"(v) : : "memory");
  return v;
}
__device__ inline int wf_keep_s(int v) {
  asm volatile("" : "+s"(v) : : "memory");
  return v;
}

// The next ticket, the same for every thread.
__device__ inline unsigned wf_take_ticket(unsigned* ctr) {
  __shared__ unsigned s_ticket;
  if (threadIdx.x == 0) s_ticket = atomicAdd(&ctr[0], 1u);
  __syncthreads();
  const unsigned t = s_ticket;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(t);
}

// Tile of ticket k in wavefront order: by m*X + Y, where m = 1 + shear, so that
// every producer of a tile -- (X-1, Y-1 .. Y+1 if sheared, else Y) and (X, Y-1)
// -- has a smaller ticket.  Column after column (X*nty + Y, which is the tile's
// index) is as good while the workgroups cover most of the front, but on a
// grid of many tile rows the 256 workgroups then cover a few columns and wait
// on each other.  512x512x64, 19-point FP64 (64 x 33 tiles):
// 1650 -> 1087 us; 256^3, 7-point FP64 (32 x 16 tiles): 320 -> 310 us.
__host__ __device__ inline long sweep_below(long d, int m, int ntx, int nty) {
  // tiles with m*X + Y < d: sum over X of d - m*X where positive, less what
  // lies beyond the last row and the last column
  auto tri = [m](long v) {
    if (v <= 0) return 0l;
    const long q = (v + m - 1) >> (m - 1);  // (m is 1 or 2)
    return q * v - ((q * (q - 1)) >> (2 - m));
  };
  const long w = (long)m * ntx;
  return tri(d) - tri(d - nty) - tri(d - w) + tri(d - w - nty);
}
__host__ __device__ inline unsigned sweep_tile(unsigned k, int sh, int ntx, int nty) {
  const int m = 1 + sh;
  int lo = 0, hi = m * (ntx - 1) + nty;  // sweep_below(lo) <= k < sweep_below(hi)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sweep_below(mid, m, ntx, nty) <= (long)k)
      lo = mid;
    else
      hi = mid;
  }
  const int r = (int)((long)k - sweep_below(lo, m, ntx, nty));
  const int x0 = lo >= nty ? (lo - nty + m) >> (m - 1) : 0;  // first X with Y = lo - m*X < nty
  const int X = x0 + r;
  return (unsigned)(X * nty + (lo - m * X));
}

// The tickets of one sweep over one grid.  A workgroup reads the buffer word
// before it takes its first ticket (the ticket's operand depends on the
// word), so whoever holds the last ticket -- the last tile's if every
// workgroup has one tile, else the last one beyond the tiles -- knows that all
// others have read it and have taken theirs, and readies counter and buffer
// word for the next launch.
struct SweepTickets {
  unsigned *ctr, *word;
  unsigned ntiles, first, par;
  bool single, started = false;
  __device__ SweepTickets(unsigned* c, unsigned* w, unsigned n) : ctr(c), word(w), ntiles(n) {
    single = ntiles <= gridDim.x;
    unsigned* s = shared();
    if (threadIdx.x == 0) {
      const unsigned p = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s[0] = p;
      s[1] = atomicAdd(&ctr[0], 1u + (p >> 31));
    }
  }
  __device__ static unsigned* shared() {
    __shared__ unsigned s[2];
    return s;
  }
  // after a barrier behind the constructor
  __device__ void start() {
    par = __builtin_amdgcn_readfirstlane(shared()[0]);
    first = __builtin_amdgcn_readfirstlane(shared()[1]);
    if (single && first == ntiles - 1u) reset();
  }
  __device__ void reset() {
    if (threadIdx.x == 0) {
      __hip_atomic_store(&ctr[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(word, par ^ 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // the next tile, the same for every thread; false: none is left
  __device__ bool take(unsigned* ticket) {
    if (started && single) return false;
    const unsigned t = started ? wf_take_ticket(ctr) : first;
    if (t >= ntiles) {  // (also a first ticket: of a workgroup that started after the others were done)
      if (t == ntiles + gridDim.x - 1u) reset();
      return false;
    }
    started = true;
    *ticket = t;
    return true;
  }
};

}  // namespace smg
