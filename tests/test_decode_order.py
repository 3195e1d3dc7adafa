"""Which unsplit calls of the decode kernel finish in the kernel: those whose u comes from workgroups that have a unit before anybody waits for it."""
import ctypes
import subprocess

import pytest

from paper_2605_08527_amd import build

SOURCE = """#include "gemm_args.h"
extern "C" int first(int tiles_m, int tiles_n, int ext, int cu_count) { return marlaas::decode_u_comes_first(tiles_m, tiles_n, ext, cu_count); }
extern "C" int column(int b, int tiles_m, int tiles_n, int ksplit, int* tm, int* ks) { int tn; marlaas::decode_tile(b, tiles_m, tiles_n, ksplit, tm, &tn, ks); return tn; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "p.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "p.hip"), "-o", str(d / "p.so")],
                   check=True, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(str(d / "p.so"))


# A unit runs one workgroup, XCD b mod 8 has an eighth of them, and workgroups get units in their order.
def test_carriers_have_units(lib):
    tm, ks = ctypes.c_int(), ctypes.c_int()
    for cus in (256, 128):
        for tiles_m in (1, 2, 3, 4, 6, 9, 17):
            for tiles_n in (8, 20, 33, 64, 65, 96, 260):
                cols = [(lib.column(b, tiles_m, tiles_n, 1, ctypes.byref(tm), ctypes.byref(ks)), tm.value) for b in range(tiles_m * tiles_n)]
                assert sorted(cols) == [(n, m) for n in range(tiles_n) for m in range(tiles_m)]
                late = {n for b, (n, _) in enumerate(cols) if b >> 3 >= cus // 8}      # column tiles with a workgroup that has to wait for a unit
                for ext in (0, 8, 32, 40, 256, 384, 1024, 4096):
                    carry = range(min(tiles_n, (ext + 31) // 32))
                    said = lib.first(tiles_m, tiles_n, ext, cus)
                    assert not said or tiles_m * tiles_n <= cus or not late.intersection(carry), (cus, tiles_m, tiles_n, ext)
                    assert said or late.intersection(carry), (cus, tiles_m, tiles_n, ext)


def test_splits_cover_their_tiles(lib):
    tm, ks = ctypes.c_int(), ctypes.c_int()
    for tiles_m, tiles_n, ksplit in ((1, 8, 8), (2, 32, 2), (2, 33, 4), (3, 7, 3), (2, 9, 16)):
        seen = {(lib.column(b, tiles_m, tiles_n, ksplit, ctypes.byref(tm), ctypes.byref(ks)), tm.value, ks.value) for b in range(tiles_m * tiles_n * ksplit)}
        assert seen == {(n, m, k) for n in range(tiles_n) for m in range(tiles_m) for k in range(ksplit)}
