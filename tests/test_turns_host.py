"""Launches that exchange u find out from lines of counters which of two areas is theirs (agent_memory.h).  The functions
themselves, compiled for the host: a workgroup's waves run one after the other between barriers, wave 0 as far ahead as it
gets, and a value that a load brings is read when it is first used, as late as a load may arrive."""
import os
import subprocess

import pytest

from paper_2605_08527_amd import build

# what the headers take from the compiler for the GPU
STUB = r"""
#pragma once
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <random>
#include <stdint.h>
#include <thread>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
typedef int hipError_t;
typedef void* hipStream_t;
struct int4 { int x, y, z, w; };
struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
struct Dim { unsigned x; };
static thread_local Dim threadIdx, blockIdx, blockDim, gridDim;
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
template <typename T> T __shfl(T v, int) { return v; }
inline uint64_t __ballot(bool b) { return b; }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
void __syncthreads();
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_readlane(x, l) (x)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __hip_atomic_compare_exchange_strong(p, old, v, o1, o2, scope) __atomic_compare_exchange_n(p, old, v, false, o1, o2)
// (asm volatile(...); is an empty statement)
#define asm
#define volatile(...)
"""

SOURCE = r"""
#include "lora_shrink.h"
using namespace marlaas;

// Waves of one workgroup, one at a time: the next one runs when this one has ended or stands at a barrier.
struct Group {
  static constexpr int WAVES = 8;
  std::mutex m;
  std::condition_variable cv;
  int now = 0, state[WAVES] = {0};                // 0: may run, 1: at a barrier, 2: ended
  void pass(int w, int s) {
    std::unique_lock<std::mutex> l(m);
    state[w] = s;
    int next = -1;
    for (int k = 0; k < WAVES && next < 0; ++k) if (state[k] == 0) next = k;
    if (next < 0)
      for (int k = 0; k < WAVES; ++k) if (state[k] == 1) { state[k] = 0; if (next < 0) next = k; }
    now = next;
    cv.notify_all();
    if (s != 2) cv.wait(l, [&] { return now == w; });
  }
};
static Group* group;
static thread_local int my_wave;
void __syncthreads() { if (group) group->pass(my_wave, 1); }

template <typename F>
static void workgroup(unsigned b, unsigned grid, F f) {
  Group g;
  group = &g;
  std::vector<std::thread> t;
  for (int w = 0; w < Group::WAVES; ++w)
    t.emplace_back([&, w] {
      my_wave = w;
      threadIdx.x = 64 * w; blockIdx.x = b; gridDim.x = grid; blockDim.x = 64 * Group::WAVES;
      { std::unique_lock<std::mutex> l(g.m); g.cv.wait(l, [&] { return g.now == w; }); }
      f(w);
      g.pass(w, 2);
    });
  for (auto& x : t) x.join();
  group = nullptr;
}

static int32_t turns[TURN_INTS];
#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// A workgroup that has its line to itself (a call of few workgroups) and no columns of its own.
int idle_workgroup() {
  for (unsigned n = 0; n < 3; ++n) {
    for (unsigned b = 0; b < 16; ++b) {
      Turn t[Group::WAVES];
      workgroup(b, 16, [&](int w) { t[w] = turn_missed(turns, 1000 + n, threadIdx.x == 0); });
      for (auto& x : t) CHECK(x.number == n && x.area == (int)(n & 1) && x.u_before == (n ? 999 + n : 0) && x.sums_ok);
    }
    for (int l = 0; l < TURN_LINES; ++l) CHECK((uint32_t)turns[l * 32] == (n + 1) << TURN_SHIFT);
  }
  return 0;
}

// A workgroup that computes u of two row blocks, its line's only one.
int producer() {
  const int64_t Kc = 512;
  std::vector<bf16_t> x(64 * Kc), L(16 * Kc);
  std::vector<f32x4> red(8 * 2 * 64);
  std::vector<float> u(64 * 16);
  ShrinkJob job = {L.data(), 1.f, 16, 0, 0, 32, 0};
  Turn t[Group::WAVES];
  bool met[Group::WAVES] = {false};
  workgroup(0, 1, [&](int w) {
    shrink_job<3, 2>(job, x.data(), Kc, Kc, 0, 0, 1, red.data(), [] {},
                     [&] {
                       const int4 l = *(const int4*)turn_line(turns);
                       const Turn was = t[w];
                       t[w] = turn_of(l.x, l.y, l.z, l.w);
                       if (met[w] && was.number != t[w].number) t[w].number = 99;
                       met[w] = true;
                       return u.data();
                     }, 16, w, 0);
    if (w == 0) turn_over(turns, t[0], 512);
  });
  CHECK(met[0] && met[1]);
  for (int w = 0; w < Group::WAVES; ++w) CHECK(!met[w] || t[w].number == 0);
  return 0;
}

// More launches than a line can number: workgroups read and add in any order, a launch's first ones when others have
// long ended; somebody gives up on the sums now and then, and always around the number's end.
int full_round() {
  std::mt19937 rng(5);
  const unsigned grids[] = {1, 2, 31, 32, 33, 64, 200};
  bool gave_before = false;
  int64_t u_before = 0;
  for (unsigned n = 0; n < 2 * (1u << (32 - TURN_SHIFT)) + 20; ++n) {
    const unsigned grid = grids[rng() % 7], number = n & (~0u >> TURN_SHIFT);
    const int64_t u = rng() % 3 ? rng() % 100000 * 4 : 0;
    std::vector<Turn> t(grid);
    std::vector<unsigned> events;                 // a workgroup's first one reads, its second one adds
    for (unsigned b = 0; b < grid; ++b) { events.push_back(b); events.push_back(b); }
    std::shuffle(events.begin(), events.end(), rng);
    std::vector<bool> seen(grid);
    bool gave = false;
    const bool may = rng() % 5 == 0 || number < 3 || number > 4092;
    for (unsigned b : events) {
      blockIdx.x = b; gridDim.x = grid;
      if (seen[b]) { turn_over(turns, t[b], u); continue; }
      seen[b] = true;
      const int4 l = *(const int4*)turn_line(turns);
      t[b] = turn_of(l.x, l.y, l.z, l.w);
      CHECK(t[b].number == number && t[b].area == (int)(n & 1) && t[b].u_before == u_before && t[b].sums_ok == !gave_before);
      if (may && t[b].sums_ok && rng() % 8 == 0) {
        for (int lane = 0; lane < 64; ++lane) turn_gave_up(turns, t[b].number, lane);
        gave = true;
      }
    }
    gave_before = gave;
    u_before = u;
  }
  return 0;
}

int main(int, char** v) {
  blockDim.x = 512;
  return !strcmp(v[1], "idle_workgroup") ? idle_workgroup() : !strcmp(v[1], "producer") ? producer() : full_round();
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("turns")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "turns.cpp").write_text("#include <algorithm>\n" + SOURCE)
    clang = os.path.join(os.path.dirname(build.HIPCC), "amdclang++")
    p = subprocess.run([clang, "-x", "c++", "-O1", "-std=c++17", "-pthread", "-w", "-I", str(d), "-I", build.CSRC, str(d / "turns.cpp"), "-o", str(d / "turns")],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    return str(d / "turns")


@pytest.mark.parametrize("what", ["idle_workgroup", "producer", "full_round"])
def test_turns(program, what):
    p = subprocess.run([program, what], stdout=subprocess.PIPE, text=True, timeout=100)
    assert p.returncode == 0, p.stdout
