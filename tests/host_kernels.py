"""Kernel sources compiled for the host: a workgroup's threads are coroutines that run one after the other.  Threads of a wave
meet where the kernel's lanes do (cross-lane operations, and inline assembly, where they must not run ahead of one
another); a wave runs as far as it gets, to a barrier or its end, before the next one starts."""
import os
import subprocess

from paper_2605_08527_amd import build

STUB = r"""
#pragma once
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <random>
#include <stdint.h>
#include <ucontext.h>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define hipLaunchKernelGGL(...) (void)0
typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0 };
inline hipError_t hipGetLastError() { return 0; }
struct int2 { int x, y; };
struct int4 { int x, y, z, w; };
struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
inline int2 make_int2(int x, int y) { return {x, y}; }
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
struct Dim { unsigned x; };
static Dim threadIdx, blockIdx, blockDim, gridDim;

// ---- one workgroup at a time
enum { RUNS, LOCKSTEP, COLLECTS, BARRIER, ENDED };
struct Thread { ucontext_t at; int state; int64_t value; std::vector<char> stack; };
static std::vector<Thread> threads;
static ucontext_t scheduler;
static int wave_size, current = -1;
static std::function<void(int)> body;
static void wait_in(int state) {
  threads[current].state = state;
  swapcontext(&threads[current].at, &scheduler);
}
static void thread_main() {
  body(current);
  threads[current].state = ENDED;
  swapcontext(&threads[current].at, &scheduler);
}
static void lockstep() { if (current >= 0) wait_in(LOCKSTEP); }
inline void __syncthreads() { wait_in(BARRIER); }
static void run_workgroup(int n, int lanes, std::function<void(int)> f) {
  threads = std::vector<Thread>(n);
  wave_size = lanes; body = f; blockDim.x = n;
  for (auto& t : threads) {
    t.stack.resize(64 << 10);
    getcontext(&t.at);
    t.at.uc_stack.ss_sp = t.stack.data(); t.at.uc_stack.ss_size = t.stack.size(); t.at.uc_link = nullptr;
    makecontext(&t.at, thread_main, 0);
    t.state = RUNS;
  }
  auto count = [&](int w, int state) { int c = 0; for (int i = w; i < w + lanes; ++i) c += threads[i].state == state; return c; };
  auto release = [&](int w, int state) { for (int i = w; i < w + lanes; ++i) if (threads[i].state == state) threads[i].state = RUNS; };
  for (bool left = true; left;) {
    left = false;
    for (int w = 0; w < n; w += lanes) {
      while (count(w, RUNS)) {
        for (int i = w; i < w + lanes; ++i)
          if (threads[i].state == RUNS) { current = i; threadIdx.x = i; swapcontext(&scheduler, &threads[i].at); }
        if (count(w, LOCKSTEP)) release(w, LOCKSTEP);
        else if (count(w, COLLECTS)) release(w, COLLECTS);
      }
      left |= count(w, BARRIER) > 0;
    }
    for (int w = 0; w < n; w += lanes) release(w, BARRIER);
  }
  current = -1;
}
// what every lane of the wave gave, once all are there (and nobody is behind)
template <typename F>
static auto collect(int64_t mine, F f) {
  threads[current].value = mine;
  wait_in(COLLECTS);
  const auto r = f(&threads[current / wave_size * wave_size]);
  wait_in(COLLECTS);
  return r;
}
inline uint64_t __ballot(bool b) {
  return collect(b, [](Thread* t) { uint64_t m = 0; for (int i = 0; i < wave_size; ++i) m |= (uint64_t)(t[i].value != 0) << i; return m; });
}
inline int __shfl_up(int v, int d) {
  const int lane = current % wave_size;
  return collect(v, [&](Thread* t) { return (int)t[lane >= d ? lane - d : lane].value; });
}
template <typename T> T __shfl(T v, int src) {
  T r = v;
  int64_t bits = 0;
  memcpy(&bits, &v, sizeof v);
  bits = collect(bits, [&](Thread* t) { return t[src % wave_size].value; });
  memcpy(&r, &bits, sizeof r);
  return r;
}

inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int atomicAdd(int* p, int v) { const int old = *p; *p += v; return old; }
inline int atomicOr(int* p, int v) { const int old = *p; *p |= v; return old; }
inline void __threadfence_system() {}
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_readlane(x, l) (x)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __hip_atomic_compare_exchange_strong(p, old, v, o1, o2, scope) __atomic_compare_exchange_n(p, old, v, false, o1, o2)
// asm volatile(...);
#define asm
#define volatile(...) lockstep()
"""


def compile_host(folder, source, flags=()):
    """The source, with the stub in place of the HIP headers, as folder/program (with -shared: a library)."""
    (folder / "hip").mkdir()
    (folder / "hip" / "hip_runtime.h").write_text(STUB)
    (folder / "source.cpp").write_text("#include <hip/hip_runtime.h>\n" + source)
    clang = os.path.join(os.path.dirname(build.HIPCC), "amdclang++")
    cmd = [clang, "-x", "c++", "-O1", "-std=c++17", "-w", "-fPIC", "-I", str(folder), "-I", build.CSRC, str(folder / "source.cpp"), "-o", str(folder / "program")]
    p = subprocess.run(cmd + list(flags), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    return str(folder / "program")
