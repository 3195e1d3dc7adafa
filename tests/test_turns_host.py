"""Launches that exchange u find out from lines of counters which of two areas is theirs (agent_memory.h).  The functions
themselves, compiled for the host: wave 0 of a workgroup runs as far ahead as it gets, and a value that a load brings is
read when it is first used, as late as a load may arrive."""
import subprocess

import pytest

from host_kernels import compile_host

SOURCE = r"""
#include "lora_shrink.h"
using namespace marlaas;

static constexpr int WAVES = 8;
// Its waves as one lane each.
template <typename F>
static void workgroup(unsigned b, unsigned grid, F f) {
  blockIdx.x = b; gridDim.x = grid;
  run_workgroup(WAVES, 1, [&](int w) { threadIdx.x = 64 * w; f(w); });
}

static int32_t turns[TURN_INTS];
#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// A workgroup that has its line to itself (a call of few workgroups) and no columns of its own.
int idle_workgroup() {
  for (unsigned n = 0; n < 3; ++n) {
    for (unsigned b = 0; b < 16; ++b) {
      Turn t[WAVES];
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
  Turn t[WAVES];
  bool met[WAVES] = {false};
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
  for (int w = 0; w < WAVES; ++w) CHECK(!met[w] || t[w].number == 0);
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
  return !strcmp(v[1], "idle_workgroup") ? idle_workgroup() : !strcmp(v[1], "producer") ? producer() : full_round();
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return compile_host(tmp_path_factory.mktemp("turns"), SOURCE)


@pytest.mark.parametrize("what", ["idle_workgroup", "producer", "full_round"])
def test_turns(program, what):
    p = subprocess.run([program, what], stdout=subprocess.PIPE, text=True, timeout=100)
    assert p.returncode == 0, p.stdout
