// What prr_topk.h needs of a GPU, on the CPU: one workgroup of 256 threads as fibers.  A wave
// operation or a barrier hands control on until every thread that takes part has come to it,
// so code whose waves reach them together behaves as on the device.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
#define __align__(n) __attribute__((aligned(n)))
#define __restrict__

struct uint4 {
  uint32_t x, y, z, w;
};
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

namespace emu {

constexpr int kThreads = 256, kLanes = 64;

struct Meet {  // where a wave's lanes, or all threads, come together
  uint64_t in[kThreads], out[kThreads];
  int arrived = 0, turn = 0;
};

struct State {
  Meet wave[kThreads / kLanes], all;
  ucontext_t main, fiber[kThreads];
  std::vector<char> stacks;
  std::function<void()> body;
  bool done[kThreads];
  int cur = 0;
  int64_t steps = 0, limit = 0;
};
inline State* S = nullptr;
struct Idx {
  struct X {
    operator int() const { return S->cur; }
  } x;
};

inline void yield() { swapcontext(&S->fiber[S->cur], &S->main); }

inline const uint64_t* meet(Meet& m, int who, int n, uint64_t v) {
  m.in[who] = v;
  ++S->steps;
  if (++m.arrived == n) {
    m.arrived = 0;
    memcpy(m.out, m.in, sizeof(m.in));
    ++m.turn;
  } else {
    const int t = m.turn;
    while (m.turn == t) yield();
  }
  return m.out;  // (valid until every one of them meets again)
}
inline const uint64_t* wave(uint64_t v) { return meet(S->wave[S->cur / kLanes], S->cur % kLanes, kLanes, v); }
inline void barrier() { meet(S->all, S->cur, kThreads, 0); }

inline void entry() {
  S->body();
  S->done[S->cur] = true;
  yield();
}

// Runs body on 256 threads; false if they have not ended after `limit` wave operations of one
// thread (counted over all of them), or if all that are left wait for ones that have ended.
inline bool run(const std::function<void()>& body, int64_t limit) {
  constexpr size_t kStack = 1 << 16;
  State s;
  S = &s;
  s.body = body;
  s.limit = limit * kThreads;
  s.stacks.resize(kStack * kThreads);
  for (int i = 0; i < kThreads; ++i) {
    s.done[i] = false;
    getcontext(&s.fiber[i]);
    s.fiber[i].uc_stack.ss_sp = s.stacks.data() + kStack * i;
    s.fiber[i].uc_stack.ss_size = kStack;
    s.fiber[i].uc_link = &s.main;
    makecontext(&s.fiber[i], entry, 0);
  }
  for (;;) {
    const int64_t before = s.steps;
    int left = 0, ended = 0;
    for (int i = 0; i < kThreads; ++i) {
      if (s.done[i]) continue;
      s.cur = i;
      swapcontext(&s.main, &s.fiber[i]);
      ++left;
      ended += s.done[i] ? 1 : 0;
    }
    if (left == 0) return true;
    if (s.steps > s.limit || (s.steps == before && ended == 0)) return false;
  }
}

}  // namespace emu

static emu::Idx threadIdx;
constexpr int kWave = emu::kLanes;

inline void __syncthreads() { emu::barrier(); }
inline uint64_t __ballot(bool p) {
  const uint64_t* v = emu::wave(p ? 1 : 0);
  uint64_t m = 0;
  for (int i = 0; i < kWave; ++i) m |= v[i] << i;
  return m;
}
inline int emu_readlane(int x, int lane) { return (int)emu::wave((uint32_t)x)[lane & 63]; }
#define __builtin_amdgcn_readlane emu_readlane
#define __builtin_amdgcn_readfirstlane(x) emu_readlane(x, 0)
#define __builtin_amdgcn_wave_barrier() ((void)emu::wave(0))
inline int __ffsll(long long x) { return __builtin_ffsll(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __clz(uint32_t x) { return x ? __builtin_clz(x) : 32; }
inline float __uint_as_float(uint32_t u) {
  float f;
  memcpy(&f, &u, 4);
  return f;
}
inline uint32_t __float_as_uint(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  return u;
}
template <class T, class V>
inline T atomicAdd(T* p, V v) {
  const T old = *p;
  *p += v;
  return old;
}
inline uint32_t atomicOr(uint32_t* p, uint32_t v) {
  const uint32_t old = *p;
  *p |= v;
  return old;
}

namespace prr {

using ::kWave;
using std::max;
using std::min;

inline int lane_id() { return emu::S->cur % kWave; }
inline int lanes_below(uint64_t m) { return __builtin_popcountll(m & ((1ull << lane_id()) - 1ull)); }
inline uint32_t score_key(float s) {
  uint32_t u = __float_as_uint(s == 0.0f ? 0.0f : s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
template <class F>
inline uint32_t wave_fold(uint32_t x, F f, int upto = kWave) {
  const uint64_t* v = emu::wave(x);
  uint32_t r = (uint32_t)v[0];
  for (int i = 1; i < upto; ++i) r = f(r, (uint32_t)v[i]);
  return r;
}
inline int wave_inclusive_scan(int x) {
  return (int)wave_fold((uint32_t)x, [](uint32_t a, uint32_t b) { return a + b; }, lane_id() + 1);
}
inline int wave_isum(int x) { return (int)wave_fold((uint32_t)x, [](uint32_t a, uint32_t b) { return a + b; }); }
inline uint32_t wave_umin(uint32_t x) { return wave_fold(x, [](uint32_t a, uint32_t b) { return a < b ? a : b; }); }
inline uint32_t wave_umax(uint32_t x) { return wave_fold(x, [](uint32_t a, uint32_t b) { return a < b ? b : a; }); }

}  // namespace prr
