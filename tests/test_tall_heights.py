"""Tall tiles of the kernel for some rows: the planner's choice against timed runs, the tiles that the GPU tests run, and sums of products followed
over all paths of the generated code."""
import ctypes
import json
import math
import os
import subprocess

import pytest

import test_gpu_tall_heights
from paper_2605_08527_amd import build
from test_generated_code import SETTLE, _functions, _registers
from test_some_rows_plan import RANKS, SOURCE as PLAN

CHOICE = PLAN[:PLAN.index("// pieces of u")].replace("int n) {", "int n, int ext, double wide) {").replace(
    "  const MidPlan p = mid_plan(T, Kc, proj, n_proj, l, 4);\n", """  int64_t all = 0;
  for (int p = 0; p < n_proj; ++p) all += cols[p];
  const MidPlan p = mid_taller(mid_plan(T, Kc, proj, n_proj, l, 4), T, Kc, proj, n_proj, l, mid_limit(T, Kc, all, ext, [&] { return wide; }));
""")


# The estimate of a tile that takes a whole unit, with 64 adapters and with 400: their producers come in rounds of units.
def test_producers_come_in_rounds(tmp_path):
    (tmp_path / "p.hip").write_text("""#include "mid_plan.h"
extern "C" double us(int n) {
  using namespace marlaas;
  ProjEntry proj[1];
  proj[0].Nout = 14336;
  MidLora l;
  l.n = n; l.tile_max = 2; l.ranks = 32 * n; l.tiles = 2 * n; l.r_stride = 32; l.tiles_max = 2 * n;
  return MidModel(512, 8192, proj, 1, l, MID_TALL).us(16, 4, 1, 0.632, 224);
}
""")
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(tmp_path / "p.hip"), "-o", str(tmp_path / "p.so")],
                   check=True, stderr=subprocess.DEVNULL)
    us = ctypes.CDLL(str(tmp_path / "p.so")).us
    us.restype = ctypes.c_double
    print("64 adapters %.1f us, 400 %.1f" % (us(64), us(400)))
    assert us(400) > us(64) + 15.0                               # (512 rows, 8192 x 14336: 153 and 228 us)


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    d = tmp_path_factory.mktemp("choice")
    (d / "p.hip").write_text(CHOICE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "p.hip"), "-o", str(d / "p.so")],
                   check=True, stderr=subprocess.DEVNULL)
    f = ctypes.CDLL(str(d / "p.so")).plan
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_double]
    return lambda T, K, cols, ranks, ext, wide: f(T, K, (ctypes.c_int32 * len(cols))(*cols), len(cols), (ctypes.c_int32 * max(len(ranks), 1))(*ranks), len(ranks), ext, wide)


def test_gpu_cases_are_what_they_say(choice):
    for name, (T, K, N, ranks) in test_gpu_tall_heights.CASES.items():
        assert choice(T, K, [N], ranks, sum(ranks), 1e9) == int(name.split(",")[0]) // 16 * 100 + 41, name
    assert [choice(T, K, [N], [], 0, 1e9) for T, K, N in test_gpu_tall_heights.WITHOUT] == [641, 841, 1041, 1641]


# 96 rows: whether producers' jobs come in two pieces, which are more workgroups than fit, or whole, does not refuse a call of fewer jobs.
def test_fewer_jobs_are_not_refused(choice):
    mixed = lambda n: [RANKS[t % 4] for t in range(n)]
    for ranks in (mixed(64), mixed(48), [32] * 64, [16] * 32, [8] * 4):          # (188, 156, 158, 47 and 19 jobs beside 240 consumers)
        assert choice(512, 5120, [5120], ranks, sum(ranks), 1e9) == 641, len(ranks)


# Against timed runs, with the weight from the memory-side cache and from memory: what the choice takes of the time without tall
# tiles, and how often it is the wrong one in either.
def test_tiles_taken(choice):
    golden = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "tall_tilings.json")))
    took = []
    for T, K, cols, n, rank, ext, wide, times in golden["sets"]:
        tile = str(choice(T, K, cols, [rank or RANKS[t % 4] for t in range(n)], ext, wide))
        took.append([a / b for a, b in zip(times.get(tile, times["small"]), times["small"])])
    for part, most in ((took[:golden["unseen"]], 0.965), (took[golden["unseen"]:], 0.955)):
        mean = math.exp(sum(math.log(q) / len(t) for t in part for q in t) / len(part))
        worst = [max(t) for t in part]
        print("%d sets, %.4f, slower by 3 %%: %d, at most %.3f" % (len(part), mean, sum(q > 1.03 for q in worst), max(worst)))
        assert mean < most and sum(q > 1.03 for q in worst) <= len(part) // 50 and max(worst) < 1.25


def _loose_sums(blocks):
    """Sums of products by inline assembly, which the compiler takes for finished at once, touched by anything but such a product
    less than SETTLE instructions behind the one that wrote them, and operands that vector arithmetic wrote less than two instructions
    before such a product, on any path."""
    order = list(blocks)
    after = dict(zip(order, order[1:]))
    state, work, found = {"": ({}, (frozenset(), frozenset()))}, [""], set()

    def reach(label, age, fresh):                    # (instructions since a sum's product; registers written one and two before)
        if label is None:
            return
        was, new = state.get(label), fresh
        if was is not None:
            age = {r: min(n, was[0].get(r, SETTLE)) for r, n in {**was[0], **age}.items()}
            new = tuple(f | w for f, w in zip(fresh, was[1]))
            if (age, new) == was:
                return
        state[label] = (dict(age), new)
        work.append(label)

    while work:
        label = work.pop()
        age, fresh = dict(state[label][0]), state[label][1]
        for s, op, operands, asm in blocks[label]:
            if op == "s_branch":
                reach(operands[0], age, fresh)
                break
            if op.startswith("s_cbranch"):
                reach(operands[0], age, fresh)
            if op == "s_endpgm":
                break
            touched = [_registers(t) for t in operands]
            ours = asm and op.startswith("v_mfma")
            if ours and any(r in f for t in touched[1:] for r in t for f in fresh):
                found.add(s)
            if not ours and any(r in age for t in touched for r in t):
                found.add(s)
            waits = int(operands[0]) + 1 if op == "s_nop" else 1
            age = {r: n + waits for r, n in age.items() if n + waits < SETTLE}
            if ours:
                age.update({r: 0 for r in touched[0]})
            wrote = frozenset(touched[0]) if op.startswith("v_") and not op.startswith("v_mfma") and touched else frozenset()
            fresh = (wrote, fresh[0]) if waits == 1 else (frozenset(), frozenset())
        else:
            reach(after.get(label), age, fresh)
    return found


def test_sums_are_settled_on_all_paths():
    out = subprocess.run([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", os.path.join(build.CSRC, "gemm_tall.hip"), "-o", "-"],
                         check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL).stdout.decode()
    kernels = list(_functions(out))
    assert len(kernels) == 4
    for name, blocks in kernels:
        assert not _loose_sums(blocks), name


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
    settled = "\ts_nop 15\n\ts_nop 15"
    for before, behind, n in (("", "", 1), ("", settled, 0), ("\tv_mov_b32_e32 v5, v1", settled, 1), ("", ".LBB0_1:", 1), ("", settled + "\n.LBB0_1:", 0),
                              ("", "\ts_cbranch_vccz .LBB0_1\n" + settled + "\n.LBB0_1:", 1), ("\tv_mov_b32_e32 v5, v1\n.LBB0_1:", settled, 1),
                              ("", "\tv_mov_b32_e32 v12, v13\n" + settled, 0)):
        (_, blocks), = _functions(text % (before, behind))
        assert len(_loose_sums(blocks)) == n, (before, behind)
