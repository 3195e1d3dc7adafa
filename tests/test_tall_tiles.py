"""Tall tiles of the kernel for some rows: where the planner takes them, and the code generated for them."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2605_08527_amd import build
from test_generated_code import SETTLE, _functions, _registers, early_moves, overwritten_reads

SOURCE = """#include "mid_plan.h"
extern "C" int taller(int64_t T, int64_t Kc, int Nout, int n, int rank, int* smaller) {
  using namespace marlaas;
  ProjEntry proj[1];
  proj[0].Nout = Nout;
  MidLora l;
  l.n = n;
  if (n) { l.tile_max = (rank + 15) / 16; l.ranks = n * rank; l.tiles = n * l.tile_max; l.r_stride = 16 * l.tile_max; l.tiles_max = l.tile_max * (n < T ? n : (int)T); }
  const MidPlan s = mid_plan(T, Kc, proj, 1, l, 4), p = mid_taller(s, T, Kc, proj, 1, l);
  *smaller = s.rb * 100 + s.wn * 10 + s.ksplit;
  const int64_t rows = 16 * p.rb;
  return p.us > s.us || p.tiles_m != (T + rows - 1) / rows ? -1 : p.rb * 100 + p.wn * 10 + p.ksplit;
}
"""


@pytest.fixture(scope="module")
def taller(tmp_path_factory):
    d = tmp_path_factory.mktemp("taller")
    (d / "p.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "p.hip"), "-o", str(d / "p.so")],
                   check=True, stderr=subprocess.DEVNULL)
    f = ctypes.CDLL(str(d / "p.so")).taller
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    return f


def test_where_they_are_taken(taller):
    """Timed: 512 rows in 240 tiles, 128, 157 and 256 rows of a wide output in 224, a square weight and a few rows in smaller ones.
    Over the whole range a plan is one of those that there are, unsplit, or the smaller one."""
    small = ctypes.c_int()
    plan = lambda *a: taller(*a, ctypes.byref(small))
    assert [plan(512, 5120, 5120, 64, 16), plan(128, 4096, 28672, 32, 16), plan(157, 4096, 28672, 32, 16), plan(256, 4096, 28672, 32, 16)] == [641, 841, 1041, 1641]
    assert plan(256, 4096, 4096, 32, 16) == small.value and plan(40, 4096, 4096, 4, 16) == small.value
    for T in (1, 17, 65, 96, 97, 129, 160, 161, 300, 511, 640, 1000, 1024):
        for K in (8, 72, 1024, 4104, 14336):
            for N in (8, 136, 2056, 10240, 14336, 28672):
                for n, rank in ((0, 0), (1, 1), (4, 128), (64, 16), (800, 8)):
                    p = plan(T, K, N, n, rank)
                    assert p == small.value or p in (641, 841, 1041, 1641), (T, K, N, n, rank, p)


def _loose_sums(blocks):
    """Sums of products by inline assembly, which the compiler takes for finished at once, touched by anything but such a product
    in a block of products, or less than SETTLE instructions behind the last one; an operand that vector arithmetic wrote right before."""
    found = []
    for instructions in blocks.values():
        since, sums, fresh = SETTLE, set(), [(), ()]
        for s, op, operands, asm in instructions:
            touched = [_registers(t) for t in operands]
            if op.startswith("v_mfma") and asm:
                if any(r in f for t in touched[1:] for r in t for f in fresh):
                    found.append(s)
                sums |= set(touched[0])
                since, fresh = 0, [(), ()]
                continue
            if since < SETTLE and any(r in sums for t in touched for r in t):
                found.append(s)
            since += int(operands[0]) + 1 if op == "s_nop" else 1
            fresh = [tuple(touched[0]) if op.startswith("v_") and touched else (), fresh[0]]
    return found


def test_code():
    """No spill, no move of a request under way, no touch of a sum before it is settled."""
    out = subprocess.run([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", os.path.join(build.CSRC, "gemm_tall.hip"), "-o", "-"],
                         check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL).stdout.decode()
    spills, counts = re.findall(r"\.vgpr_spill_count: +(\d+)", out), [int(n) for n in re.findall(r"\.vgpr_count: +(\d+)", out)]
    assert spills == ["0"] * 4 and counts[0] <= 128 and max(counts) <= 256
    for name, blocks in _functions(out):
        assert not early_moves(blocks) and not overwritten_reads(blocks) and not _loose_sums(blocks), name


def test_loose_sum_is_seen():
    text = """_Zk:
%s
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]
\t;;#ASMEND
%s
\tds_write_b128 v20, v[0:3]
\ts_endpgm
.Lfunc_end0:
"""
    for before, behind, n in (("", "", 1), ("", "\ts_nop 15\n\ts_nop 15", 0), ("\tv_mov_b32_e32 v5, v1", "\ts_nop 15\n\ts_nop 15", 1)):
        (_, blocks), = _functions(text % (before, behind))
        assert len(_loose_sums(blocks)) == n, (before, behind)
