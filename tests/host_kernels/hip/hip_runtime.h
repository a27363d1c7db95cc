// Host stand-in for the HIP names that the pass kernels use: one workgroup at
// a time, its lanes as cooperating fibers of one OS thread.  A lane runs until
// it meets a workgroup barrier or a cross-lane exchange; lanes that have
// returned do not hold a barrier up (the hardware counts live waves only).
// Workgroup memory belongs to the thread, so it keeps what the last workgroup
// left there, as LDS does.  Between two barriers or exchanges a lane runs by
// itself, so lanes that relied on running in step would be found out.
#pragma once
#include <ucontext.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ thread_local
#define __align__(n) __attribute__((aligned(n)))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))

struct HostDim {
  unsigned x, y, z;
};
inline HostDim threadIdx{0, 0, 0}, blockIdx{0, 0, 0}, blockDim{1, 1, 1}, gridDim{1, 1, 1};

namespace hostgpu {

enum State { READY, AT_BLOCK, AT_WAVE, ENDED };
struct Lane {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  State state = READY;
};
inline std::vector<Lane>* lanes = nullptr;
inline ucontext_t scheduler;
inline int current = 0;
inline const std::function<void()>* body = nullptr;
alignas(16) inline char wave_slot[64][16];

inline void yield(State s) {
  Lane& l = (*lanes)[current];
  l.state = s;
  swapcontext(&l.ctx, &scheduler);
}
inline void entry() {
  (*body)();
  (*lanes)[current].state = ENDED;
  swapcontext(&(*lanes)[current].ctx, &scheduler);
}

// Run one workgroup of n lanes, its waves in the order given; before_wave(i)
// is called before the i-th wave of that order first runs.
inline void run_block(int n, const std::vector<int>& order, const std::function<void()>& f,
                      const std::function<void(int)>& before_wave) {
  std::vector<Lane> ls(n);
  lanes = &ls;
  body = &f;
  blockDim = {(unsigned)n, 1, 1};
  for (int i = 0; i < n; ++i) {
    ls[i].stack.reset(new char[1 << 17]);
    getcontext(&ls[i].ctx);
    ls[i].ctx.uc_stack.ss_sp = ls[i].stack.get();
    ls[i].ctx.uc_stack.ss_size = 1 << 17;
    ls[i].ctx.uc_link = nullptr;
    makecontext(&ls[i].ctx, entry, 0);
  }
  // a wave's lanes run until each has ended or waits at the workgroup barrier
  auto run_wave = [&](int w) {
    const int lo = 64 * w, hi = std::min(n, lo + 64);
    for (;;) {
      bool ran = false;
      for (int i = lo; i < hi; ++i) {
        if (ls[i].state != READY) continue;
        ran = true;
        current = i;
        threadIdx = {(unsigned)i, 0, 0};
        swapcontext(&scheduler, &ls[i].ctx);
      }
      if (ran) continue;
      bool released = false;
      for (int i = lo; i < hi; ++i)
        if (ls[i].state == AT_WAVE) {
          ls[i].state = READY;
          released = true;
        }
      if (!released) return;
    }
  };
  bool first = true;
  for (;;) {
    for (int i = 0; i < (int)order.size(); ++i) {
      if (first) before_wave(i);
      run_wave(order[i]);
    }
    first = false;
    bool waiting = false;
    for (Lane& l : ls)
      if (l.state == AT_BLOCK) {
        l.state = READY;
        waiting = true;
      }
    if (!waiting) return;
  }
}

template <typename T>
T exchange(T v, int src) {
  static_assert(sizeof(T) <= 16, "lane slot");
  std::memcpy(wave_slot[current & 63], &v, sizeof(T));
  yield(AT_WAVE);
  T out;
  std::memcpy(&out, wave_slot[src], sizeof(T));
  yield(AT_WAVE);
  return out;
}

}  // namespace hostgpu

#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_wave_barrier() hostgpu::yield(hostgpu::AT_WAVE)

struct int4 {
  int x, y, z, w;
};
template <typename T>
constexpr T min(T a, T b) {
  return b < a ? b : a;
}

inline void __syncthreads() { hostgpu::yield(hostgpu::AT_BLOCK); }
template <typename T>
T __shfl(T v, int src, int) {
  return hostgpu::exchange(v, src & 63);
}
template <typename T>
T __shfl_down(T v, int off, int) {
  const int lane = hostgpu::current & 63;
  return hostgpu::exchange(v, lane + off < 64 ? lane + off : lane);
}
