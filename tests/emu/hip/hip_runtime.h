// A CPU stand-in for what the sweep kernels use of HIP, so that their own
// source runs on the host (tests/test_sweep_emulation.py compiles it with
// clang++, the inline assembly taken out).
//
// A workgroup is an OS thread, its lanes are fibers of that thread.  A lane
// runs until a barrier, an operation across its wave (ballot, DPP) or a sleep;
// the lanes of a workgroup take turns in an order drawn from a seed, so that
// what lies between two barriers runs in many orders.  Workgroups run
// concurrently and see each other's stores.  Buffer accesses are range-checked
// as the hardware does, and against the arrays the test registered.
#pragma once
#include <math.h>
#include <sched.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <atomic>
#include <functional>
#include <thread>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) alignas(n)
#define __shared__ static thread_local

typedef _Float16 __half;
typedef void* hipStream_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum { hipFuncAttributeMaxDynamicSharedMemorySize = 0 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace emu {

enum State { RUN, BARRIER, WAVE, DONE };
struct Fiber {
  ucontext_t ctx;
  dim3 tid;
  State state;
  uint64_t give, take[64];  // an operation across the wave: this lane's value, every lane's
};
struct Group {
  std::vector<Fiber> f;
  ucontext_t main;
  Fiber* cur = nullptr;
  dim3 block, grid, dim;
  unsigned char* dyn = nullptr;
  const std::function<void()>* body = nullptr;
};
inline thread_local Group* G = nullptr;

struct Range {
  const char *lo, *hi;
};
inline std::vector<Range> arrays;          // registered device arrays
inline std::atomic<int> errors{0};
inline unsigned cap = 0;                   // workgroups of a persistent kernel (0: as launched)
inline bool plain = false;                 // kernels without barriers: lanes as plain calls
inline uint64_t seed = 1;

inline void error(const char* what) {
  if (errors.fetch_add(1) < 5) fprintf(stderr, "emulation: %s\n", what);
}
inline void yield(State s) {
  if (plain) {
    error("a barrier in a plain kernel");
    abort();
  }
  G->cur->state = s;
  swapcontext(&G->cur->ctx, &G->main);
}
inline const uint64_t* wave(uint64_t v) {
  Fiber* me = G->cur;
  me->give = v;
  yield(WAVE);
  return me->take;
}
inline void sleep() {
  sched_yield();
  yield(RUN);
}
inline void entry() {
  (*G->body)();
  G->cur->state = DONE;
  swapcontext(&G->cur->ctx, &G->main);
}
inline void check(const void* p, size_t n) {
  for (const Range& r : arrays)
    if ((const char*)p >= r.lo && (const char*)p + n <= r.hi) return;
  error("access outside the arrays");
}

// The lanes of one workgroup until all are done.
inline void run_group(Group& g, uint64_t rng) {
  const size_t stack = 96 * 1024, n = g.f.size();
  char* const mem = (char*)mmap(nullptr, stack * n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  G = &g;
  std::vector<unsigned> order(n);
  for (unsigned i = 0; i < n; ++i) {
    Fiber& f = g.f[i];
    f.tid = dim3(i, 0, 0);
    f.state = RUN;
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = mem + stack * i;
    f.ctx.uc_stack.ss_size = stack;
    f.ctx.uc_link = &g.main;
    makecontext(&f.ctx, entry, 0);
    order[i] = i;
  }
  for (;;) {
    // waves in a drawn order, lanes of a wave in turn or in reverse
    rng = rng * 6364136223846793005ull + 1442695040888963407ull;
    const unsigned waves = (unsigned)(n + 63) / 64, w0 = (unsigned)(rng >> 33) % waves;
    const bool up = (rng >> 62) & 1, lane_up = (rng >> 61) & 1;
    bool ran = false, alive = false;
    for (unsigned k = 0; k < waves; ++k) {
      const unsigned w = (up ? w0 + k : w0 + waves - k) % waves;
      for (unsigned l = 0; l < 64; ++l) {
        const unsigned i = w * 64 + (lane_up ? l : 63 - l);
        if (i >= n || g.f[i].state != RUN) continue;
        ran = true;
        g.cur = &g.f[i];
        swapcontext(&g.main, &g.f[i].ctx);
      }
    }
    bool barrier = true;
    for (const Fiber& f : g.f) {
      alive |= f.state != DONE;
      barrier &= f.state == BARRIER || f.state == DONE;
    }
    if (!alive) break;
    bool moved = ran;
    if (barrier) {
      for (Fiber& f : g.f)
        if (f.state == BARRIER) f.state = RUN;
      moved = true;
    }
    for (unsigned w = 0; w < waves; ++w) {
      bool all = true, any = false;
      const unsigned i0 = w * 64, i1 = i0 + 64 < n ? i0 + 64 : (unsigned)n;
      for (unsigned i = i0; i < i1; ++i) {
        any |= g.f[i].state == WAVE;
        all &= g.f[i].state == WAVE || g.f[i].state == DONE;
      }
      if (!any || !all) continue;
      for (unsigned i = i0; i < i1; ++i) {
        for (unsigned j = i0; j < i1; ++j) g.f[i].take[j - i0] = g.f[j].state == WAVE ? g.f[j].give : 0;
      }
      for (unsigned i = i0; i < i1; ++i)
        if (g.f[i].state == WAVE) g.f[i].state = RUN;
      moved = true;
    }
    if (!moved) {
      error("lanes wait at different barriers");
      abort();
    }
  }
  munmap(mem, stack * n);
}

// Memory whose end (rounded to 16 bytes) is followed by a page that faults.
inline char* guarded(size_t bytes, int fill) {
  const size_t pg = 4096, use = (bytes + 15) / 16 * 16, len = (use + pg - 1) / pg * pg;
  char* m = (char*)mmap(nullptr, len + pg, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  mprotect(m + len, pg, PROT_NONE);
  memset(m, fill, len);
  return m + len - use;
}
inline void unguard(char* p, size_t bytes) {
  const size_t pg = 4096, use = (bytes + 15) / 16 * 16, len = (use + pg - 1) / pg * pg;
  munmap(p + use - len, len + pg);
}

inline void launch(dim3 grid, dim3 dim, size_t lds, const std::function<void()>& body) {
  if (cap != 0 && !plain && grid.x > cap) grid.x = cap;
  auto group = [&](unsigned b) {
    Group g;
    g.block = dim3(b, 0, 0);
    g.grid = grid;
    g.dim = dim;
    g.body = &body;
    if (plain) {
      g.f.resize(1);
      G = &g;
      g.cur = &g.f[0];
      for (unsigned t = 0; t < dim.x; ++t) {
        g.f[0].tid = dim3(t, 0, 0);
        body();
      }
      return;
    }
    g.f.resize(dim.x);
    if (lds) g.dyn = (unsigned char*)guarded(lds, 0xff);
    run_group(g, seed * 7919 + b);
    if (lds) unguard((char*)g.dyn, lds);
  };
  if (plain) {
    for (unsigned b = 0; b < grid.x; ++b) group(b);
    return;
  }
  std::vector<std::thread> t;
  for (unsigned b = 0; b < grid.x; ++b) t.emplace_back(group, b);
  for (auto& x : t) x.join();
}

struct Buffer {
  const char* p;
  unsigned n;
};
template <class T>
inline T load(Buffer r, unsigned off, unsigned soff) {
  T v;
  memset(&v, 0, sizeof v);
  if ((uint64_t)off + soff + sizeof(T) > r.n) return v;
  check(r.p + off + soff, sizeof(T));
  memcpy(&v, r.p + off + soff, sizeof v);
  return v;
}
template <class T>
inline void store(T v, Buffer r, unsigned off, unsigned soff) {
  if ((uint64_t)off + soff + sizeof(T) > r.n) return;
  check(r.p + off + soff, sizeof(T));
  memcpy(const_cast<char*>(r.p) + off + soff, &v, sizeof v);
}

template <class U>
inline U atomic_load(const U* p) {
  check(p, sizeof(U));
  return __atomic_load_n(p, __ATOMIC_SEQ_CST);
}
template <class U>
inline void atomic_store(U* p, U v) {
  check(p, sizeof(U));
  __atomic_store_n(p, v, __ATOMIC_SEQ_CST);
}
inline uint64_t ballot(bool v) {
  const uint64_t* t = wave(v);
  uint64_t r = 0;
  for (unsigned i = 0; i < 64; ++i) r |= (uint64_t)(t[i] != 0) << i;
  return r;
}
inline int quad(int v, int ctrl) {
  const unsigned lane = G->cur->tid.x % 64;
  return (int)wave((unsigned)v)[(lane & ~3u) + (ctrl & 3)];
}

// float(half M of w) times sc, rounded once
inline float half_times(unsigned w, int m, float sc) {
  const unsigned short u = (unsigned short)(m ? w >> 16 : w);
  __half h;
  memcpy(&h, &u, 2);
  return (float)h * sc;
}

}  // namespace emu

#define threadIdx (emu::G->cur->tid)
#define blockIdx (emu::G->block)
#define gridDim (emu::G->grid)
#define blockDim (emu::G->dim)
#define __syncthreads() emu::yield(emu::BARRIER)
#define hipLaunchKernelGGL(K, GRID, BLOCK, LDS, STREAM, ...) emu::launch(GRID, BLOCK, LDS, [&] { K(__VA_ARGS__); })
#define EMU_DYN_LDS (emu::G->dyn)

typedef unsigned emu_u2 __attribute__((ext_vector_type(2)));
typedef unsigned emu_u4 __attribute__((ext_vector_type(4)));
typedef emu::Buffer __amdgpu_buffer_rsrc_t;
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, n, flags) (emu::Buffer{(const char*)(p), (unsigned)(n)})
#define __builtin_amdgcn_raw_buffer_load_b32(r, o, s, c) emu::load<unsigned>(r, o, s)
#define __builtin_amdgcn_raw_buffer_load_b64(r, o, s, c) emu::load<emu_u2>(r, o, s)
#define __builtin_amdgcn_raw_buffer_load_b128(r, o, s, c) emu::load<emu_u4>(r, o, s)
#define __builtin_amdgcn_raw_buffer_store_b32(v, r, o, s, c) emu::store<unsigned>(v, r, o, s)
#define __builtin_amdgcn_raw_buffer_store_b64(v, r, o, s, c) emu::store<emu_u2>(v, r, o, s)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_ballot_w64(v) emu::ballot(v)
#define __builtin_amdgcn_mov_dpp(v, c, a, b, d) emu::quad(v, c)
#define __builtin_amdgcn_s_sleep(n) emu::sleep()
#define __builtin_amdgcn_s_setprio(n) ((void)0)
#define __builtin_amdgcn_sched_barrier(n) ((void)0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, o, s) emu::atomic_load(p)
#define __hip_atomic_store(p, v, o, s) emu::atomic_store(p, v)
inline unsigned atomicAdd(unsigned* p, unsigned v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
inline unsigned atomicOr(unsigned* p, unsigned v) { return __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }

template <class T, class F>
inline T emu_cast(F f) {
  return __builtin_bit_cast(T, f);
}
inline long long __double_as_longlong(double v) { return emu_cast<long long>(v); }
inline double __longlong_as_double(long long v) { return emu_cast<double>(v); }
inline unsigned __float_as_uint(float v) { return emu_cast<unsigned>(v); }
inline float __uint_as_float(unsigned v) { return emu_cast<float>(v); }
inline int __float_as_int(float v) { return emu_cast<int>(v); }
inline float __int_as_float(int v) { return emu_cast<float>(v); }
inline double __shfl_down(double v, int off, int) {
  const unsigned lane = threadIdx.x % 64;
  return emu_cast<double>(emu::wave(emu_cast<uint64_t>(v))[lane + off < 64 ? lane + off : lane]);
}
inline float __half2float(__half v) { return (float)v; }
inline __half __float2half_rn(float v) { return (__half)v; }
inline __half __ushort_as_half(unsigned short v) { return emu_cast<__half>(v); }
inline unsigned short __half_as_ushort(__half v) { return emu_cast<unsigned short>(v); }
