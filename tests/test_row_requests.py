"""Which calls request their operands a row at a time, against timed runs of both."""
import ctypes
import subprocess

import pytest

from paper_2605_08527_amd import build

SOURCE = """#include "lora_shrink.h"
extern "C" int few(int64_t T, int64_t Kc, int64_t lda) { return marlaas::thin_rows(T, Kc, lda); }
extern "C" int job(int64_t Kc, int S, int rows, int workgroups) { return marlaas::shrink_rows(Kc, S, rows, workgroups); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "p.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "p.hip"), "-o", str(d / "p.so")],
                   check=True, stderr=subprocess.DEVNULL)
    so = ctypes.CDLL(str(d / "p.so"))
    so.few.argtypes = [ctypes.c_int64] * 3
    so.job.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return so


# (rows, contraction, distance of the rows) that took 1.5 % longer and more with such requests, and 3 % less and more
def test_few_rows(lib):
    assert not any(lib.few(T, K, K) for T, K in ((1, 2600), (1, 14336), (2, 2000), (2, 14336), (4, 2600), (4, 7000), (8, 2600), (8, 7464), (9, 6152), (10, 2600), (12, 1024), (16, 2000), (20, 2000)))
    assert all(lib.few(T, K, K) for T, K in ((8, 8192), (10, 5120), (12, 8192), (14, 14336), (16, 4096), (18, 3072), (24, 5120), (32, 2600), (32, 4096)))
    assert lib.few(16, 8192, 8192) and not lib.few(16, 8192, 8200) and lib.few(16, 8184, 9216)


# producers' jobs: few rows of an adapter, however long the contraction, four steps a wave and launches of many workgroups do without
def test_jobs(lib):
    assert not any(lib.job(*j) for j in ((1864, 1, 3, 300), (4112, 1, 8, 300), (14336, 2, 1, 300), (1024, 1, 32, 300), (4096, 4, 32, 300), (4096, 1, 32, 641)))
    assert not any(lib.job(*j) for j in ((5120, 1, 4, 300), (5120, 2, 8, 300), (4544, 1, 8, 300), (5120, 1, 8, 641)))
    assert all(lib.job(*j) for j in ((5120, 1, 5, 428), (4608, 1, 8, 300)))
    assert all(lib.job(*j) for j in ((1056, 1, 9, 300), (4096, 2, 16, 300), (14336, 4, 32, 640)))
