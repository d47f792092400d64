// Runs HIP kernels on the CPU, so that a sanitizer sees every memory access
// of theirs.  A source file that includes this instead of the HIP headers
// compiles with clang++ as plain C++: address spaces are dropped, LDS arrays
// are statics, and the lanes of a workgroup are fibers that meet at barriers
// and at the wave's cross-lane operations.  One workgroup runs at a time, in
// an order that Options::seed shuffles.  Lanes of a wave that wait at
// different places stop the program: no kernel here may do that.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <random>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define address_space(n)

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};

namespace cpu {

struct Options {
  unsigned seed = 0;              // order of a launch's workgroups, contents of new device memory
  size_t largest = SIZE_MAX;      // an allocation above this fails
  size_t allocated = 0;           // by the last one that did not
};
inline Options options;

enum Op : int { kBallot, kShfl, kShflUp, kShflXor, kFirst, kSync };
enum State : int { kRun, kWave, kBlock, kDone };
struct Lane {
  void* sp;
  State state;
  Op op;
  uint64_t value;
  unsigned arg;
  uint64_t result;
};

inline std::vector<Lane> lanes;
struct Stacks : std::vector<void*> {
  ~Stacks() {
    for (void* s : *this) free(s);
  }
};
inline Stacks stacks;
constexpr size_t kStack = 1 << 18;
inline unsigned current;
inline void* scheduler_sp;
inline const std::function<void()>* body;
inline dim3 block_idx, grid_dim, block_dim;

extern "C" void cpu_fiber_switch(void** from, void* to);
__asm__(
    ".text\n.globl cpu_fiber_switch\n.type cpu_fiber_switch,@function\ncpu_fiber_switch:\n"
    "pushq %rbp\npushq %rbx\npushq %r12\npushq %r13\npushq %r14\npushq %r15\n"
    "movq %rsp,(%rdi)\nmovq %rsi,%rsp\n"
    "popq %r15\npopq %r14\npopq %r13\npopq %r12\npopq %rbx\npopq %rbp\nret\n"
    ".size cpu_fiber_switch,.-cpu_fiber_switch\n");

[[noreturn]] inline void stop(const char* why) {
  fprintf(stderr, "workgroup %u: %s\n", block_idx.x, why);
  exit(4);
}
inline void leave(State s) {
  Lane& l = lanes[current];
  l.state = s;
  cpu_fiber_switch(&l.sp, scheduler_sp);
}
inline void lane_main() {
  (*body)();
  leave(kDone);
  abort();
}
inline uint64_t wave_op(Op op, uint64_t value, unsigned arg = 0) {
  Lane& l = lanes[current];
  l.op = op;
  l.value = value;
  l.arg = arg;
  leave(kWave);
  return lanes[current].result;
}

// The wave whose lanes all wait at the same operation.
inline void finish_wave(unsigned w0, unsigned n) {
  uint64_t live = 0, votes = 0;
  unsigned first = 64;
  for (unsigned i = 0; i < n; ++i) {
    const Lane& l = lanes[w0 + i];
    if (l.state == kDone) continue;
    if (first == 64) first = i;
    if (l.op != lanes[w0 + first].op) stop("lanes of a wave wait at different operations");
    live |= uint64_t{1} << i;
    if (l.value) votes |= uint64_t{1} << i;
  }
  for (unsigned i = 0; i < n; ++i) {
    Lane& l = lanes[w0 + i];
    if (l.state == kDone) continue;
    unsigned from = i;
    switch (l.op) {
      case kBallot: l.result = votes; break;
      case kFirst: l.result = lanes[w0 + first].value; break;
      case kSync: break;
      case kShfl: from = l.arg & 63u; break;
      case kShflUp: from = i >= l.arg ? i - l.arg : i; break;
      case kShflXor: from = i ^ l.arg; break;
    }
    if (l.op == kShfl || l.op == kShflUp || l.op == kShflXor) {
      if (from >= n || !(live >> from & 1)) stop("a lane reads a lane that has left");
      l.result = lanes[w0 + from].value;
    }
    l.state = kRun;
  }
}

inline void run_workgroup(unsigned threads) {
  lanes.assign(threads, Lane{});
  while (stacks.size() < threads) stacks.push_back(aligned_alloc(64, kStack));
  for (unsigned t = 0; t < threads; ++t) {
    void** top = reinterpret_cast<void**>(static_cast<char*>(stacks[t]) + kStack) - 2;
    *top = reinterpret_cast<void*>(&lane_main);
    lanes[t].sp = top - 6;
    memset(lanes[t].sp, 0, 6 * sizeof(void*));
  }
  for (;;) {
    bool moved = false, all_done = true;
    unsigned at_barrier = 0, live = 0;
    for (unsigned w0 = 0; w0 < threads; w0 += 64) {
      const unsigned n = std::min(64u, threads - w0);
      unsigned waiting = 0, here = 0;
      for (unsigned i = 0; i < n; ++i) {
        current = w0 + i;
        if (lanes[current].state == kRun) {
          cpu_fiber_switch(&scheduler_sp, lanes[current].sp);
          moved = true;
        }
        const State s = lanes[w0 + i].state;
        here += s != kDone;
        waiting += s == kWave;
        at_barrier += s == kBlock;
      }
      live += here;
      if (waiting && waiting == here) {
        finish_wave(w0, n);
        moved = true;
      }
      all_done = all_done && here == 0;
    }
    if (all_done) return;
    if (at_barrier == live) {
      for (Lane& l : lanes)
        if (l.state == kBlock) l.state = kRun;
      moved = true;
    }
    if (!moved) stop("its lanes wait for each other");
  }
}

inline bool launch(dim3 grid, dim3 block, const std::function<void()>& f) {
  if (grid.x == 0 || block.x == 0 || block.x > 1024 || uint64_t{grid.x} * block.x > 0xFFFFFFFFu) return false;
  body = &f;
  grid_dim = grid;
  block_dim = block;
  std::vector<unsigned> order(grid.x);
  for (unsigned i = 0; i < grid.x; ++i) order[i] = i;
  if (options.seed) std::shuffle(order.begin(), order.end(), std::mt19937(options.seed));
  for (unsigned b : order) {
    block_idx = dim3(b);
    run_workgroup(block.x);
  }
  return true;
}

struct ThreadIdx {
  struct X {
    operator unsigned() const { return current; }
  } x;
};
inline ThreadIdx thread_idx;

// Called with the name of each kernel that is launched.
inline std::function<void(const char*)> before_launch = [](const char*) {};

}  // namespace cpu

#define threadIdx (cpu::thread_idx)
#define blockIdx (cpu::block_idx)
#define gridDim (cpu::grid_dim)
#define blockDim (cpu::block_dim)

inline void __syncthreads() { cpu::leave(cpu::kBlock); }
inline uint64_t __ballot(bool p) { return cpu::wave_op(cpu::kBallot, p); }
inline int __shfl(int v, int lane) { return static_cast<int>(cpu::wave_op(cpu::kShfl, static_cast<uint32_t>(v), static_cast<unsigned>(lane))); }
inline int __shfl_up(int v, unsigned d) { return static_cast<int>(cpu::wave_op(cpu::kShflUp, static_cast<uint32_t>(v), d)); }
inline int __shfl_xor(int v, int d) { return static_cast<int>(cpu::wave_op(cpu::kShflXor, static_cast<uint32_t>(v), static_cast<unsigned>(d))); }

inline int cpu_readfirstlane(int v) { return static_cast<int>(cpu::wave_op(cpu::kFirst, static_cast<uint32_t>(v))); }
inline void cpu_wave_barrier() { cpu::wave_op(cpu::kSync, 0); }
// Byte i of the result is byte (sel's byte i) of b (0-3) or a (4-7); 12 gives
// 0x00, above it 0xFF.
inline uint32_t cpu_perm(uint32_t a, uint32_t b, uint32_t sel) {
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = sel >> (8 * i) & 0xFFu;
    if (s >= 8 && s < 12) cpu::stop("a byte permute that repeats a sign");
    r |= (s < 4 ? b >> (8 * s) & 0xFFu : s < 8 ? a >> (8 * (s - 4)) & 0xFFu : s == 12 ? 0u : 0xFFu) << (8 * i);
  }
  return r;
}
inline uint32_t cpu_alignbit(uint32_t hi, uint32_t lo, uint32_t sh) {
  return static_cast<uint32_t>((static_cast<uint64_t>(hi) << 32 | lo) >> (sh & 31u));
}
inline uint32_t cpu_mbcnt(uint32_t mask, uint32_t add, unsigned first) {
  const unsigned lane = cpu::current & 63u;
  const uint64_t below = lane <= first ? 0 : lane >= first + 32 ? 0xFFFFFFFFull : (uint64_t{1} << (lane - first)) - 1;
  return add + static_cast<uint32_t>(__builtin_popcountll(mask & below));
}
#define __builtin_amdgcn_readfirstlane cpu_readfirstlane
#define __builtin_amdgcn_wave_barrier cpu_wave_barrier
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_perm cpu_perm
#define __builtin_amdgcn_alignbit cpu_alignbit
#define __builtin_amdgcn_mbcnt_lo(m, a) cpu_mbcnt(m, a, 0)
#define __builtin_amdgcn_mbcnt_hi(m, a) cpu_mbcnt(m, a, 32)
#define __HIP_MEMORY_SCOPE_WAVEFRONT 0
#define __hip_atomic_fetch_add(p, v, order, scope) cpu_fetch_add(p, v)

template <class T, class V>
inline T cpu_fetch_add(T* p, V v) {
  const T was = *p;
  *p = was + static_cast<T>(v);
  return was;
}
template <class T>
inline T atomicAdd(T* p, T v) { return cpu_fetch_add(p, v); }
template <class T>
inline T atomicMin(T* p, T v) {
  const T was = *p;
  *p = v < was ? v : was;
  return was;
}
template <class T>
inline T atomicExch(T* p, T v) {
  const T was = *p;
  *p = v;
  return was;
}
template <class T>
inline T atomicCAS(T* p, T expected, T v) {
  const T was = *p;
  if (was == expected) *p = v;
  return was;
}

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidConfiguration = 9 };
enum { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
inline hipError_t cpu_last_error = hipSuccess;

template <class T>
inline hipError_t hipMalloc(T** p, size_t bytes) {
  if (bytes > cpu::options.largest) return cpu_last_error = hipErrorOutOfMemory;
  cpu::options.allocated = bytes;
  uint8_t* d = static_cast<uint8_t*>(aligned_alloc(256, bytes));
  if (!d) return hipErrorOutOfMemory;
  std::mt19937 rng(cpu::options.seed + 1);
  for (size_t i = 0; i < bytes; ++i) d[i] = static_cast<uint8_t>(rng());  // device memory holds anything
  *p = reinterpret_cast<T*>(d);
  return hipSuccess;
}
inline hipError_t hipFree(void* p) {
  free(p);
  return hipSuccess;
}
inline hipError_t hipMemcpy(void* to, const void* from, size_t bytes, int) {
  memcpy(to, from, bytes);
  return hipSuccess;
}
inline hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipGetLastError() {
  const hipError_t e = cpu_last_error;
  cpu_last_error = hipSuccess;
  return e;
}
inline const char* hipGetErrorString(hipError_t) { return "error"; }
template <class F>
inline hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, F, int, size_t) {
  *n = 1;
  return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, shared, stream, ...) \
  (void)(stream), cpu::before_launch(#kernel), (void)(cpu::launch(grid, block, [&] { kernel(__VA_ARGS__); }) || (cpu_last_error = hipErrorInvalidConfiguration))
