"""The tiling that the planner of the kernel for some rows takes, against timed runs of every tiling."""
import ctypes
import json
import math
import os
import subprocess

import pytest

from paper_2605_08527_amd import build

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "some_rows_tilings.json")
RANKS = (8, 16, 32, 64)

SOURCE = """#include "mid_plan.h"
#include <functional>
#include <vector>
extern "C" int plan(int64_t T, int64_t Kc, const int32_t* cols, int n_proj, const int32_t* ranks, int n) {
  using namespace marlaas;
  ProjEntry proj[8];
  for (int p = 0; p < n_proj; ++p) proj[p].Nout = cols[p];
  MidLora l;
  l.n = n;
  for (int t = 0; t < n; ++t) {
    const int tiles = (ranks[t] + 15) / 16;
    l.ranks += ranks[t]; l.tiles += tiles; l.tile_max = std::max(l.tile_max, tiles); l.r_stride = std::max(l.r_stride, 16 * tiles);
  }
  std::vector<int> by_size;
  for (int t = 0; t < n; ++t) by_size.push_back((ranks[t] + 15) / 16);
  std::sort(by_size.begin(), by_size.end(), std::greater<int>());
  for (int t = 0; t < n && t < T; ++t) l.tiles_max += by_size[t];
  const MidPlan p = mid_plan(T, Kc, proj, n_proj, l, 4);
  return p.rb * 100 + p.wn * 10 + p.ksplit;
}
// pieces of u, -1: more of it than an area holds
extern "C" int pieces(int64_t T, int64_t Kc, int n_proj, int r_stride, int64_t consumers, int64_t jobs) {
  const int64_t u = T * r_stride * n_proj;
  const int s = marlaas::mid_u_splits(Kc, u, marlaas::MID_U_FLOATS, consumers, jobs, 256);
  return s * u > marlaas::MID_U_FLOATS ? -1 : s;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "plan.hip"), "-o", str(d / "plan.so")],
                   check=True, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(str(d / "plan.so"))


@pytest.fixture(scope="module")
def excess(lib):
    """(a set's values, time of the tiling taken over the best one's)"""
    plan = lib.plan
    plan.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_int]
    out = []
    for T, K, cols, n, rank, times in json.load(open(GOLDEN))["sets"]:
        ranks = [rank or RANKS[t % 4] for t in range(n)]
        taken = plan(T, K, (ctypes.c_int32 * len(cols))(*cols), len(cols), (ctypes.c_int32 * max(n, 1))(*ranks), n)
        out.append(((T, K, n), times[str(taken)] / min(times.values())))
    return out


def _mean(values):
    return math.exp(sum(math.log(v) for v in values) / len(values))


# The runs of a set differ by about 1 %, and no rule of a few terms finds the best of twelve tilings every time.
def test_tilings_taken(excess):
    assert len(excess) == 425
    print("all %.4f, without adapters %.4f, contractions up to 2048 %.4f, at most %.3f" % (
        _mean([q for _, q in excess]), _mean([q for (_, _, n), q in excess if n == 0]), _mean([q for (_, K, _), q in excess if K <= 2048]), max(q for _, q in excess)))
    assert _mean([q for _, q in excess]) < 1.026
    assert _mean([q for (_, _, n), q in excess if n == 0]) < 1.02
    assert max(q for _, q in excess) < 1.35


# Contractions too long for a whole producer are cut, however much u there is: up to eight projections, 1024 rows, rank 128.
@pytest.mark.parametrize("n_proj", [1, 3, 5, 8])
@pytest.mark.parametrize("T,K", [(600, 6400), (1000, 14336), (1024, 8192)])
def test_long_contractions_are_cut(lib, n_proj, T, K):
    f = lib.pieces
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    for r_stride in (16, 64, 112, 128):
        assert f(T, K, n_proj, r_stride, 1024, 4096) == 2
