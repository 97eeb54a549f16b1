// One workgroup of a HIP kernel on the host: every thread is a fiber, and a
// thread runs until it reaches a shuffle (which needs its wavefront) or a
// barrier (which needs the workgroup).  Of the threads that can run, those of
// the first wavefront in `order` go first, so that each order of the
// wavefronts that the barriers allow can be tried: a missing barrier gives a
// wrong result in some order, every time.
#pragma once

#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(x)
#define __shared__ static

struct Dim1 {
  unsigned x;
};
static Dim1 threadIdx{0}, blockIdx{0}, blockDim{256}, gridDim{1};

namespace emu {

enum State { kReady, kWave, kBlockWait, kDone };

constexpr int kThreads = 256, kWaves = kThreads / 64;
static ucontext_t g_main, g_ctx[kThreads];
static State g_state[kThreads];
static std::vector<char> g_stack[kThreads];
static unsigned long long g_slot[2][kThreads];
static int g_parity[kThreads];
static std::function<void()> g_body;

static void yield(State s) {
  const int t = (int)threadIdx.x;
  g_state[t] = s;
  swapcontext(&g_ctx[t], &g_main);
}

static void entry() {
  g_body();
  g_state[threadIdx.x] = kDone;
}

// Run the workgroup; false if it cannot finish (a barrier or a shuffle that
// not all threads reach).
static bool run(const int order[kWaves], std::function<void()> body) {
  g_body = body;
  for (int t = 0; t < kThreads; ++t) {
    g_stack[t].resize(1 << 16);
    getcontext(&g_ctx[t]);
    g_ctx[t].uc_stack.ss_sp = g_stack[t].data();
    g_ctx[t].uc_stack.ss_size = g_stack[t].size();
    g_ctx[t].uc_link = &g_main;
    makecontext(&g_ctx[t], entry, 0);
    g_state[t] = kReady;
    g_parity[t] = 0;
  }
  for (;;) {
    int next = -1, at_block = 0, done = 0;
    for (int w = 0; w < kWaves && next < 0; ++w) {
      int at_wave = 0;
      for (int l = 0; l < 64; ++l) at_wave += g_state[64 * order[w] + l] == kWave;
      for (int l = 0; l < 64; ++l) {
        State& s = g_state[64 * order[w] + l];
        if (at_wave == 64) s = kReady;
        if (s == kReady && next < 0) next = 64 * order[w] + l;
        at_block += s == kBlockWait;
        done += s == kDone;
      }
    }
    if (next < 0) {
      if (done == kThreads) return true;
      if (at_block != kThreads) return false;
      for (int t = 0; t < kThreads; ++t) g_state[t] = kReady;
      continue;
    }
    threadIdx.x = (unsigned)next;
    swapcontext(&g_main, &g_ctx[next]);
  }
}

}  // namespace emu

inline void __syncthreads() { emu::yield(emu::kBlockWait); }

inline unsigned long long __shfl_xor(unsigned long long v, int o, int) {
  const int t = (int)threadIdx.x, b = emu::g_parity[t];
  emu::g_parity[t] ^= 1;
  emu::g_slot[b][t] = v;
  emu::yield(emu::kWave);
  return emu::g_slot[b][t ^ o];
}

inline long long __double_as_longlong(double v) {
  long long r;
  std::memcpy(&r, &v, 8);
  return r;
}

inline double __longlong_as_double(long long v) {
  double r;
  std::memcpy(&r, &v, 8);
  return r;
}

inline int atomicExch(int* p, int v) {
  const int old = *p;
  *p = v;
  return old;
}
