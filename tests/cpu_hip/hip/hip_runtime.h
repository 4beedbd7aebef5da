// The part of HIP that lossy.hip and serialize.hip use, for building them as
// plain C++ in tests: kernels run block by block on the CPU, every thread a
// fiber that yields at barriers and at the exchanges of its wave.  Launches
// run at once; `after_launch` lets a test act between two launches of a call,
// as another stream would.
#pragma once
#include <math.h>
#include <setjmp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) ((void*)&(x))

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct __attribute__((aligned(16))) float4 { float x, y, z, w; };
struct __attribute__((aligned(8))) float2 { float x, y; };
struct __attribute__((aligned(8))) uint2 { unsigned x, y; };
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice = 101, hipErrorInvalidSymbol = 13 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipGetSymbolAddress(void** p, void* s) { return *p = s, hipSuccess; }

namespace cpu_hip {

inline dim3 g_thread, g_block, g_block_dim, g_grid_dim;
inline std::function<void(const char*)> after_launch;

enum State { kReady, kWave, kBlock, kDone };
struct Fiber {
  ucontext_t start;
  jmp_buf at;
  std::vector<char> stack;
  bool started;
  State state;
};
struct Block {
  std::vector<Fiber> fibers;
  std::vector<uint64_t> slot;  // a wave exchange's values, one per thread
  jmp_buf scheduler;
  const std::function<void()>* body;
};
inline Block g_run;

__attribute__((noinline)) inline void wait(State s) {
  Fiber& f = g_run.fibers[g_thread.x];
  f.state = s;
  if (!_setjmp(f.at)) _longjmp(g_run.scheduler, 1);
}

inline void entry() {
  (*g_run.body)();
  g_run.fibers[g_thread.x].state = kDone;
  _longjmp(g_run.scheduler, 1);
}

inline void run_block(unsigned threads, const std::function<void()>& body) {
  std::vector<Fiber>& fs = g_run.fibers;
  if (fs.size() < threads) fs.resize(threads);
  g_run.slot.resize(fs.size());
  g_run.body = &body;
  for (unsigned t = 0; t < threads; t++) fs[t].state = kReady, fs[t].started = false;
  for (;;) {
    for (volatile unsigned t = 0; t < threads; t = t + 1) {
      Fiber& f = fs[t];
      if (f.state != kReady) continue;
      g_thread.x = t;
      if (_setjmp(g_run.scheduler)) continue;
      if (f.started) _longjmp(f.at, 1);
      f.started = true;
      f.stack.resize(65536);
      getcontext(&f.start);
      f.start.uc_stack.ss_sp = f.stack.data();
      f.start.uc_stack.ss_size = f.stack.size();
      f.start.uc_link = nullptr;
      makecontext(&f.start, entry, 0);
      setcontext(&f.start);
    }
    unsigned done = 0, block = 0, woken = 0;
    for (unsigned w = 0; w < threads; w += 64) {
      const unsigned end = w + 64 < threads ? w + 64 : threads;
      unsigned wave = 0, live = 0;
      for (unsigned t = w; t < end; t++) {
        live += fs[t].state != kDone;
        wave += fs[t].state == kWave;
        block += fs[t].state == kBlock;
        done += fs[t].state == kDone;
      }
      if (live && wave == live)
        for (unsigned t = w; t < end; t++)
          if (fs[t].state == kWave) fs[t].state = kReady, woken++;
    }
    if (done == threads) return;
    if (!woken) {
      if (block + done != threads) fprintf(stderr, "threads wait at different places\n"), abort();
      for (unsigned t = 0; t < threads; t++)
        if (fs[t].state == kBlock) fs[t].state = kReady;
    }
  }
}

inline void launch(const char* name, dim3 grid, dim3 block, const std::function<void()>& body) {
  g_grid_dim = grid;
  g_block_dim = block;
  for (unsigned b = 0; b < grid.x; b++) {
    g_block.x = b;
    run_block(block.x, body);
  }
  if (after_launch) after_launch(name);
}

template <class T>
T exchange(T v, unsigned src) {
  static_assert(sizeof(T) <= 8, "");
  memcpy(&g_run.slot[g_thread.x], &v, sizeof(T));
  wait(kWave);
  T r;
  memcpy(&r, &g_run.slot[(g_thread.x & ~63u) + src], sizeof(T));
  wait(kWave);
  return r;
}

inline uint64_t ballot(bool p) {
  g_run.slot[g_thread.x] = p;
  wait(kWave);
  uint64_t r = 0;
  const unsigned w = g_thread.x & ~63u;
  for (unsigned l = 0; l < 64 && w + l < g_block_dim.x; l++)
    if (g_run.fibers[w + l].state != kDone && g_run.slot[w + l]) r |= 1ull << l;
  wait(kWave);
  return r;
}

}  // namespace cpu_hip

#define threadIdx cpu_hip::g_thread
#define blockIdx cpu_hip::g_block
#define blockDim cpu_hip::g_block_dim
#define gridDim cpu_hip::g_grid_dim
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
  cpu_hip::launch(#kernel, grid, block, [&] { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { cpu_hip::wait(cpu_hip::kBlock); }
template <class T>
T __shfl_xor(T v, int m) {
  return cpu_hip::exchange(v, (threadIdx.x & 63) ^ m);
}
template <class T>
T __shfl_down(T v, int d) {
  const unsigned l = threadIdx.x & 63;
  return cpu_hip::exchange(v, l + d < 64 ? l + d : l);
}
template <class T>
T __shfl_up(T v, int d) {
  const int l = threadIdx.x & 63;
  return cpu_hip::exchange(v, l >= d ? l - d : l);
}
template <class T>
T __shfl(T v, int l) {
  return cpu_hip::exchange(v, l & 63);
}
#define __builtin_amdgcn_readlane(v, l) __shfl(v, l)
inline uint64_t __ballot(bool p) { return cpu_hip::ballot(p); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline unsigned atomicAdd(unsigned* p, unsigned v) {
  const unsigned old = *p;
  *p += v;
  return old;
}
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline uint32_t __float_as_uint(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  return u;
}
