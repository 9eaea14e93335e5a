// Kernels on the CPU, for checks of their barriers and addresses: a stand-in for
// the HIP header that lets g++ compile the kernel sources as they are.  A
// workgroup's threads are fibers of one host thread, each run until it waits at
// a barrier (or a wave operation, which exchanges values between the 64 lanes of
// a wave); the wave that goes first after a barrier runs up to the next one
// before any other moves, in an order the caller picks, so that a missing wait
// gives a wrong result every time.  Waves that wait at a barrier for lanes of
// their own that have ended, and workgroups that wait for ever, are errors.
// Launches and runtime calls in the sources compile to nothing.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <random>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ thread_local
#define __forceinline__ inline
#define __launch_bounds__(...)

using std::isnan;
using std::max;
using std::min;

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct alignas(16) double2 {
  double x, y;
};
struct alignas(16) float4 {
  float x, y, z, w;
};
struct alignas(16) uint4 {
  unsigned x, y, z, w;
};
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace emu {

enum State { READY, AT_BARRIER, AT_WAVE, DONE };
struct Fiber {
  ucontext_t ctx;
  State state = READY;
  std::vector<char> stack;
};
inline std::vector<Fiber> fibers;
inline std::vector<uint64_t> lane_value;
inline ucontext_t scheduler;
inline unsigned current = 0;
inline std::function<void()> body;

inline void wait(State s) {
  Fiber& f = fibers[current];
  f.state = s;
  swapcontext(&f.ctx, &scheduler);
}

inline void enter() {
  body();
  fibers[current].state = DONE;
  swapcontext(&fibers[current].ctx, &scheduler);
}

inline void fail(const char* what) {
  printf("workgroup %u: %s\n", blockIdx.x, what);
  exit(3);
}

enum Order { ASCENDING, DESCENDING, RANDOM };

// every workgroup of a launch, one after another
inline void launch(dim3 grid, unsigned threads, Order order, const std::function<void()>& kernel) {
  static std::mt19937 rng(3);
  body = kernel;
  gridDim = grid;
  blockDim = dim3(threads);
  const unsigned waves = (threads + 63) / 64;
  std::vector<unsigned> turn(waves);
  for (unsigned w = 0; w < waves; w++) turn[w] = order == DESCENDING ? waves - 1 - w : w;
  for (unsigned b = 0; b < grid.x * grid.y; b++) {
    blockIdx = dim3(b % grid.x, b / grid.x, 0);
    fibers.resize(threads);
    lane_value.assign(waves * 64, 0);
    for (unsigned t = 0; t < threads; t++) {
      Fiber& f = fibers[t];
      f.state = READY;
      f.stack.resize(64 << 10);
      getcontext(&f.ctx);
      f.ctx.uc_stack.ss_sp = f.stack.data();
      f.ctx.uc_stack.ss_size = f.stack.size();
      f.ctx.uc_link = &scheduler;
      makecontext(&f.ctx, enter, 0);
    }
    for (;;) {
      if (order == RANDOM) std::shuffle(turn.begin(), turn.end(), rng);
      unsigned done = 0, waiting = 0;
      for (unsigned w : turn) {
        const unsigned t0 = 64 * w, t1 = std::min(threads, t0 + 64);
        for (bool again = true; again;) {
          unsigned at_wave = 0, ended = 0;
          for (unsigned t = t0; t < t1; t++) {
            if (fibers[t].state == READY) {
              current = t;
              threadIdx = dim3(t, 0, 0);
              swapcontext(&scheduler, &fibers[t].ctx);
            }
            at_wave += fibers[t].state == AT_WAVE;
            ended += fibers[t].state == DONE;
          }
          again = at_wave > 0;
          if (at_wave && at_wave + ended != t1 - t0) fail("lanes of a wave at a barrier and at a wave operation");
          if (!at_wave && ended && ended != t1 - t0) fail("lanes of a wave ended while others wait at a barrier");
          if (at_wave)
            for (unsigned t = t0; t < t1; t++)
              if (fibers[t].state == AT_WAVE) fibers[t].state = READY;
        }
        for (unsigned t = t0; t < t1; t++) {
          done += fibers[t].state == DONE;
          waiting += fibers[t].state == AT_BARRIER;
        }
      }
      if (done == threads) break;
      if (done) fail("waves ended while others wait at a barrier");
      for (Fiber& f : fibers) f.state = READY;
    }
  }
}

// a value of another lane of the wave
template <class T>
T from_lane(T v, unsigned lane) {
  uint64_t q = 0;
  memcpy(&q, &v, sizeof v);
  lane_value[current] = q;
  wait(AT_WAVE);
  q = lane_value[(current & ~63u) + (lane & 63)];
  wait(AT_WAVE);
  memcpy(&v, &q, sizeof v);
  return v;
}

}  // namespace emu

inline void __syncthreads() { emu::wait(emu::AT_BARRIER); }
template <class T>
T __shfl(T v, int lane, int = 64) {
  return emu::from_lane(v, (unsigned)lane);
}
template <class T>
T __shfl_xor(T v, int mask, int = 64) {
  return emu::from_lane(v, (emu::current & 63u) ^ (unsigned)mask);
}
inline int __any(int p) {
  for (int o = 32; o > 0; o >>= 1) p |= __shfl_xor(p != 0, o);
  return p;
}
template <class T>
T atomicAdd(T* p, T v) {
  const T old = *p;
  *p = old + v;
  return old;
}
template <class T>
T atomicMax(T* p, T v) {
  const T old = *p;
  *p = v > old ? v : old;
  return old;
}
template <class T>
T atomicOr(T* p, T v) {
  const T old = *p;
  *p = old | v;
  return old;
}
inline void __threadfence() {}
inline void __threadfence_block() {}
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __clz(int x) { return x ? __builtin_clz((unsigned)x) : 32; }
template <class To, class From>
To bits_as(From v) {
  To r;
  memcpy(&r, &v, sizeof r);
  return r;
}
inline double __longlong_as_double(long long v) { return bits_as<double>(v); }
inline long long __double_as_longlong(double v) { return bits_as<long long>(v); }
inline float __uint_as_float(unsigned v) { return bits_as<float>(v); }
inline unsigned __float_as_uint(float v) { return bits_as<unsigned>(v); }
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_s_getreg(x) 0u
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() emu::wait(emu::AT_WAVE)

typedef struct Stream* hipStream_t;
enum hipError_t { hipSuccess, hipErrorInvalidValue, hipErrorUnknown };
inline hipError_t hipGetLastError() { return hipSuccess; }
#define hipLaunchKernelGGL(...) ((void)0)

// the runtime calls of the sources' host code: never reached
typedef struct Graph* hipGraph_t;
typedef struct GraphExec* hipGraphExec_t;
typedef struct Event* hipEvent_t;
enum {
  hipStreamCaptureModeThreadLocal,
  hipMemcpyDeviceToDevice,
  hipMemcpyDeviceToHost,
  hipMemcpyHostToDevice,
  hipFuncAttributeMaxDynamicSharedMemorySize
};
inline const char* hipGetErrorString(hipError_t) { return "no GPU"; }
#define EMU_NO_GPU(name)             \
  template <class... A>              \
  inline hipError_t name(A&&...) {   \
    return hipErrorUnknown;          \
  }
EMU_NO_GPU(hipStreamBeginCapture)
EMU_NO_GPU(hipStreamEndCapture)
EMU_NO_GPU(hipStreamSynchronize)
EMU_NO_GPU(hipGraphInstantiate)
EMU_NO_GPU(hipGraphLaunch)
EMU_NO_GPU(hipGraphDestroy)
EMU_NO_GPU(hipGraphExecDestroy)
EMU_NO_GPU(hipEventCreate)
EMU_NO_GPU(hipEventRecord)
EMU_NO_GPU(hipEventDestroy)
EMU_NO_GPU(hipEventElapsedTime)
EMU_NO_GPU(hipMemcpyAsync)
EMU_NO_GPU(hipMemsetAsync)
EMU_NO_GPU(hipFuncSetAttribute)
EMU_NO_GPU(hipHostMalloc)
EMU_NO_GPU(hipHostFree)
