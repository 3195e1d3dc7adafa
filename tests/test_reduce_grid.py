"""The grid of the weight gradients' reductions for very unequal segments stays inside what a launch takes."""
import ctypes
import subprocess

import pytest

from paper_2605_08527_amd import build

SOURCE = """#include "common.h"
extern "C" int rows(int64_t T, int n, const int32_t* len) {
  const int chunk = marlaas::reduce_ragged_chunk(T, n);
  int slots = 0;
  for (int t = 0; t < n; ++t) {
    const int pieces = (len[t] + chunk - 1) / chunk;
    if (pieces > 1) slots += pieces;
  }
  return marlaas::reduce_ragged_rows(n, slots);
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "rows.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "rows.hip"), "-o", str(d / "rows.so")],
                   check=True, stderr=subprocess.DEVNULL)
    f = ctypes.CDLL(str(d / "rows.so")).rows
    return lambda lens: f(ctypes.c_int64(sum(lens)), len(lens), (ctypes.c_int32 * len(lens))(*lens))


# one adapter with half of all rows among hundreds that are just cut; as many as there can be; a few; none is cut
@pytest.mark.parametrize("lens", [[262144] + [513] * 500 + [3] * 1547, [500000] + [513] * 1000 + [0] * 3095, [2 ** 30] + [2 ** 18] * 4095,
                                  [600] * 4096, [5000, 1], [100] * 64])
def test_rows_of_the_grid(rows, lens):
    got, n = rows(lens), len(lens)
    chunk = (max(512, 2 * sum(lens) // n) + 63) // 64 * 64
    pieces = sum(-(-v // chunk) for v in lens if v > chunk)
    assert got == n + pieces
    assert got < 3 * n and got <= 65535
