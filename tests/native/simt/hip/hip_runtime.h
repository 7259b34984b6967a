// hip_runtime.h - a host stand-in for the HIP runtime, for tests only: runs a
// kernel's source on the CPU, so that what waves and workgroups do to each
// other can be looked at in orders that a GPU seldom takes.
//
// A lane is a fiber.  The lanes of a wave go on together from one cross-lane
// operation to the next (all lanes of the wave have to reach it); which wave
// of a workgroup goes on next is drawn at every such operation and at every
// atomic one.  The workgroups of a launch run one after another, or, for launches
// of simt::concurrent workgroups, side by side in threads.
#pragma once

#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <random>
#include <thread>
#include <type_traits>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static thread_local
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 1
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct int2 { int32_t x, y; };
struct int4 { int32_t x, y, z, w; };
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };

typedef int hipError_t;
typedef struct simt_stream* hipStream_t;
typedef struct simt_event* hipEvent_t;
typedef struct simt_graph* hipGraphExec_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
enum { hipHostMallocDefault = 0, hipStreamNonBlocking = 1, hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
inline const char* hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = nullptr;
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
template <class T>
inline hipError_t hipHostMalloc(T** p, size_t n, unsigned) {
  *p = static_cast<T*>(std::malloc(n));
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
template <class T>
inline hipError_t hipMalloc(T** p, size_t n) {
  *p = static_cast<T*>(std::malloc(n));
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}

namespace simt {

struct Block;
struct Lane {
  void* sp = nullptr;   // saved stack pointer while it does not run
  Block* block = nullptr;
  dim3 tid;
  bool ready = false, done = false;
};
struct Wave {
  std::vector<Lane*> lanes;
  uint64_t buf[2][64];
  uint64_t mask[2] = {0, 0};   // lanes that took part
  int arrived = 0, live = 0;
  uint32_t gen = 0;
};
struct Block {
  std::vector<Lane> lanes;
  std::vector<Wave> waves;
  std::mt19937_64 rng;
  void* sp = nullptr;     // the scheduler's
  int arrived = 0, live = 0;
  dim3 idx, dim, grid;
  const std::function<void()>* body = nullptr;
};

inline thread_local Lane* cur = nullptr;
inline unsigned concurrent = 0;      // launches of this many workgroups run them in threads
inline unsigned grid_now = 0;        // workgroups of the launch that runs
inline uint64_t seed = 1;
inline uint64_t hold = 1;            // most turns that a lane waits before an atomic operation
// Called by a lane before an atomic operation (a test may hold it up there).
inline void (*on_atomic)(unsigned block, unsigned thread) = nullptr;
// Launches until one fails (0: none does): it does not run.
inline int fail_launch = 0;
inline int last_error = 0;
// Called when the host waits for a stream.
inline void (*on_sync)() = nullptr;

// Saves the callee's registers on this stack, keeps its pointer in *from and
// goes on with the stack `to`.
extern "C" void simt_switch(void** from, void* to);
asm(R"(
.text
.weak simt_switch
.type simt_switch,@function
simt_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
.size simt_switch,.-simt_switch
)");

inline Wave& wave_of(Lane* l) { return l->block->waves[l->tid.x >> 6]; }
inline void leave() {
  simt_switch(&cur->sp, cur->block->sp);
}
inline void wake_wave(Wave& w) {
  w.arrived = 0;
  ++w.gen;
  w.mask[w.gen & 1] = 0;
  for (Lane* l : w.lanes)
    if (!l->done) l->ready = true;
}
inline void wake_block(Block& b) {
  b.arrived = 0;
  for (Lane& l : b.lanes)
    if (!l.done) l.ready = true;
}

// All lanes of the wave bring a value; returns the slots and the lanes.
inline const uint64_t* exchange(uint64_t v, uint64_t* mask = nullptr) {
  Lane* me = cur;
  Wave& w = wave_of(me);
  const uint32_t g = w.gen & 1, lane = me->tid.x & 63;
  w.buf[g][lane] = v;
  w.mask[g] |= 1ull << lane;
  if (++w.arrived == w.live) {
    const uint64_t keep = w.mask[g];
    wake_wave(w);
    w.mask[g] = keep;
    w.mask[w.gen & 1] = 0;
  } else {
    me->ready = false;
  }
  leave();
  if (mask) *mask = w.mask[g];
  return w.buf[g];
}
inline void sync_block() {
  Lane* me = cur;
  Block& b = *me->block;
  if (++b.arrived == b.live) {
    wake_block(b);
  } else {
    me->ready = false;
  }
  leave();
}
inline void finish_lane() {
  Lane* me = cur;
  Block& b = *me->block;
  Wave& w = wave_of(me);
  me->done = true;
  me->ready = false;
  --b.live;
  if (--w.live > 0 && w.arrived == w.live) wake_wave(w);
  if (b.live > 0 && b.arrived == b.live) wake_block(b);
  leave();
}
inline void lane_main() {
  (*cur->block->body)();
  finish_lane();
  std::abort();
}
inline void atomic_point() {
  if (!cur) return;
  if (on_atomic) on_atomic(cur->block->idx.x, cur->tid.x);
  auto& rng = cur->block->rng;
  for (uint64_t n = 1 + (rng() & 1 ? rng() % hold : 0); n > 0; --n) leave();   // stays ready
}

inline void run_block(dim3 idx, dim3 grid, dim3 dim, const std::function<void()>& body, uint64_t s) {
  Block b;
  b.rng.seed(s);
  b.idx = idx;
  b.dim = dim;
  b.grid = grid;
  b.body = &body;
  b.lanes.resize(dim.x);
  b.waves.resize((dim.x + 63) / 64);
  b.live = (int)dim.x;
  constexpr size_t kStack = 64 << 10;
  char* stacks = static_cast<char*>(mmap(nullptr, kStack * dim.x, PROT_READ | PROT_WRITE,
                                         MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
  if (stacks == MAP_FAILED) std::abort();
  for (unsigned t = 0; t < dim.x; ++t) {
    Lane& l = b.lanes[t];
    l.block = &b;
    l.tid = dim3(t, 0, 0);
    l.ready = true;
    b.waves[t >> 6].lanes.push_back(&l);
    ++b.waves[t >> 6].live;
    auto** top = reinterpret_cast<void**>(stacks + kStack * (t + 1)) - 2;
    *--top = nullptr;                                // where lane_main would return to
    *--top = reinterpret_cast<void*>(&lane_main);
    for (int i = 0; i < 6; ++i) *--top = nullptr;
    l.sp = top;
  }
  std::vector<unsigned> open;
  while (b.live > 0) {
    open.clear();
    for (unsigned w = 0; w < b.waves.size(); ++w)
      for (Lane* l : b.waves[w].lanes)
        if (l->ready) {
          open.push_back(w);
          break;
        }
    if (open.empty()) {
      std::fprintf(stderr, "simt: workgroup %u: lanes wait for each other\n", idx.x);
      std::exit(3);
    }
    Wave& w = b.waves[open[b.rng() % open.size()]];
    for (Lane* l : w.lanes)
      if (l->ready) {
        cur = l;
        simt_switch(&b.sp, l->sp);
        cur = nullptr;
      }
  }
  munmap(stacks, kStack * dim.x);
}

inline void launch(dim3 grid, dim3 dim, const std::function<void()>& body) {
  if (fail_launch > 0 && --fail_launch == 0) {
    last_error = hipErrorOutOfMemory;
    return;
  }
  grid_now = grid.x;
  if (grid.x != concurrent) {
    for (unsigned i = 0; i < grid.x; ++i) run_block(dim3(i, 0, 0), grid, dim, body, seed * 1000003u + i);
    return;
  }
  std::vector<std::thread> th;
  for (unsigned i = 0; i < grid.x; ++i)
    th.emplace_back([=, &body] { run_block(dim3(i, 0, 0), grid, dim, body, seed * 1000003u + i); });
  for (auto& t : th) t.join();
}

}  // namespace simt

inline hipError_t hipStreamSynchronize(hipStream_t) {
  if (simt::on_sync) simt::on_sync();
  return hipSuccess;
}

inline hipError_t hipGetLastError() {
  const hipError_t e = simt::last_error;
  simt::last_error = hipSuccess;
  return e;
}
#define threadIdx (simt::cur->tid)
#define blockIdx (simt::cur->block->idx)
#define blockDim (simt::cur->block->dim)
#define gridDim (simt::cur->block->grid)
#define hipLaunchKernelGGL(kern, grid, block, lds, stream, ...) \
  simt::launch(grid, block, [&] { kern(__VA_ARGS__); })

// ---- cross-lane operations ----------------------------------------------------

inline unsigned __lane_id() { return threadIdx.x & 63u; }
inline uint64_t __ballot(bool p) {
  uint64_t mask;
  const uint64_t* b = simt::exchange(p ? 1 : 0, &mask);
  uint64_t r = 0;
  for (int i = 0; i < 64; ++i)
    if ((mask >> i) & 1u) r |= (b[i] & 1u) << i;
  return r;
}
inline int __builtin_amdgcn_readlane(int x, int lane) { return (int)simt::exchange((uint32_t)x)[lane & 63]; }
inline int __builtin_amdgcn_readfirstlane(int x) {
  uint64_t mask;
  const uint64_t* b = simt::exchange((uint32_t)x, &mask);
  return (int)b[__builtin_ctzll(mask)];
}
inline int __shfl(int x, int lane, int = 64) { return (int)simt::exchange((uint32_t)x)[lane & 63]; }
inline int __shfl_xor(int x, int m, int = 64) {
  const int lane = (int)(threadIdx.x & 63u);
  return (int)simt::exchange((uint32_t)x)[lane ^ m];
}
inline int __shfl_up(int x, int d, int = 64) {
  const int lane = (int)(threadIdx.x & 63u);
  return (int)simt::exchange((uint32_t)x)[lane >= d ? lane - d : lane];
}
inline int __shfl_down(int x, int d, int = 64) {
  const int lane = (int)(threadIdx.x & 63u);
  return (int)simt::exchange((uint32_t)x)[lane + d < 64 ? lane + d : lane];
}
// row_shr 1 to 15 (0x111 ..), row_bcast 15 and 31 (0x142, 0x143), as the
// reductions use them; a lane without a source, or of a masked row, keeps old.
inline int __builtin_amdgcn_update_dpp(int old, int x, int ctrl, int row_mask, int, bool) {
  const int lane = (int)(threadIdx.x & 63u), row = lane >> 4;
  const uint64_t* b = simt::exchange((uint32_t)x);
  int src = -1;
  if (ctrl >= 0x111 && ctrl <= 0x11f) src = (lane & 15) >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
  else if (ctrl == 0x142) src = row > 0 ? row * 16 - 1 : -1;
  else if (ctrl == 0x143) src = row > 1 ? 31 : -1;
  else std::abort();
  return src >= 0 && ((row_mask >> row) & 1) ? (int)b[src] : old;
}
inline unsigned __builtin_amdgcn_mbcnt_lo(unsigned m, unsigned x) {
  const unsigned lane = threadIdx.x & 63u;
  return x + (unsigned)__builtin_popcount(lane < 32 ? m & ((1u << lane) - 1u) : m);
}
inline unsigned __builtin_amdgcn_mbcnt_hi(unsigned m, unsigned x) {
  const unsigned lane = threadIdx.x & 63u;
  return x + (lane < 32 ? 0u : (unsigned)__builtin_popcount(m & ((1u << (lane - 32)) - 1u)));
}
inline void __builtin_amdgcn_wave_barrier() { simt::exchange(0); }
#define __builtin_amdgcn_fence(order, scope) __atomic_thread_fence(__ATOMIC_SEQ_CST)
inline void __builtin_amdgcn_s_waitcnt(int) { __atomic_thread_fence(__ATOMIC_SEQ_CST); }
inline void __threadfence() { __atomic_thread_fence(__ATOMIC_SEQ_CST); }
inline void __threadfence_block() { simt::exchange(0); }
inline void __syncthreads() { simt::sync_block(); }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }

// ---- atomics --------------------------------------------------------------------

template <class T> struct simt_same { typedef T type; };
#define SIMT_ATOMIC(name, expr)                                              \
  template <class T>                                                         \
  inline T name(T* p, typename simt_same<T>::type v) {                       \
    simt::atomic_point();                                                    \
    T old = __atomic_load_n(p, __ATOMIC_SEQ_CST);                            \
    while (!__atomic_compare_exchange_n(p, &old, (T)(expr), false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {} \
    return old;                                                              \
  }
SIMT_ATOMIC(atomicAdd, old + v)
SIMT_ATOMIC(atomicSub, old - v)
SIMT_ATOMIC(atomicMin, old < v ? old : v)
SIMT_ATOMIC(atomicMax, old > v ? old : v)
SIMT_ATOMIC(atomicOr, old | v)
SIMT_ATOMIC(atomicAnd, old & v)
SIMT_ATOMIC(atomicExch, v)
template <class T>
inline T atomicCAS(T* p, typename simt_same<T>::type expect, typename simt_same<T>::type v) {
  simt::atomic_point();
  T old = expect;
  __atomic_compare_exchange_n(p, &old, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return old;
}
template <class T>
inline T __hip_atomic_load(const T* p, int, int) {
  return __atomic_load_n(p, __ATOMIC_SEQ_CST);
}
template <class T>
inline void __hip_atomic_store(T* p, typename simt_same<T>::type v, int, int) {
  __atomic_store_n(p, v, __ATOMIC_SEQ_CST);
}

template <class A, class B>
inline typename std::common_type<A, B>::type min(A a, B b) {
  typedef typename std::common_type<A, B>::type T;
  return (T)a < (T)b ? (T)a : (T)b;
}
template <class A, class B>
inline typename std::common_type<A, B>::type max(A a, B b) {
  typedef typename std::common_type<A, B>::type T;
  return (T)a < (T)b ? (T)b : (T)a;
}
