"""Operands that are requested a row at a time and put in order through LDS, on both sides of the lines from which that is done:
contractions that end inside a 32-deep step, and with waves that have fewer steps than others or none."""
import numpy as np
import pytest

from harness import workloads as wl
from paper_2605_08527_amd import api
from helpers import HipLayer, assert_close, to_host

pytestmark = pytest.mark.gpu


# x of few rows: more than eight of them, more than eight 32-deep steps a wave (2048)
@pytest.mark.parametrize("T", [8, 9, 16, 17, 32])
@pytest.mark.parametrize("K", [2048, 2056, 2088, 4104])
def test_few_rows(oracle, T, K):
    _check(oracle, T, K, 72, [16, 8, 24])


# around the lines themselves: more than eight steps a wave from 17 rows on, before that rows 2 KB apart and more than 192 rows times steps
@pytest.mark.parametrize("T,K", [(1, 14336), (7, 8192), (8, 6144), (8, 7168), (12, 4096), (13, 4096), (13, 4104), (16, 3072), (16, 5120), (17, 2048), (17, 2056), (32, 2056)])
def test_few_rows_around_the_line(oracle, T, K):
    _check(oracle, T, K, 72, [16, 8, 24])
    _check(oracle, T, K, 4168, [16])


# u of batches with few rows for a compute unit, in a launch of its own
@pytest.mark.parametrize("K,ranks", [(2048, [16]), (2056, [8, 24, 32]), (2088, [64, 40]), (2056, [128, 100]), (4104, [16, 9])])
def test_shrink_of_few_rows_a_unit(oracle, K, ranks):
    _check(oracle, 1030, K, 4104, ranks, packed=False)


@pytest.mark.parametrize("K,ranks", [(2816, [16]), (2824, [8, 24, 32]), (2824, [64, 40]), (2856, [128, 100])])
def test_shrink_around_its_line(oracle, K, ranks):
    _check(oracle, 1030, K, 4104, ranks, packed=False)


# u of some more rows, by producers beside the consumers: more than four steps a wave (from a contraction of 1032 on where it is not cut), two
# blocks of rows and one, rows of others in them, ranks that leave rows of the factor out
@pytest.mark.parametrize("T", [33, 100, 257])
@pytest.mark.parametrize("K,ranks", [(1024, [16]), (1032, [16]), (1032, [8, 24, 9] * 8), (2072, [64, 40, 16] * 4), (4104, [16] * 6), (4136, [128, 100])])
def test_producers_of_some_rows(oracle, T, K, ranks):
    _check(oracle, T, K, 1096, ranks)


def _check(oracle, T, K, N, ranks, packed=True):
    ids = np.random.default_rng(T * K).integers(-1, len(ranks), size=T).astype(np.int32)
    w = wl.make_layer(T + K, T, K, N, ranks, [0.5 + t for t in range(len(ranks))], ids, dtype="bf16", layout=wl.TORCH)
    L = HipLayer(w, table=True, packed=packed)
    api.marlaas_profile_enable(L.ctx, True)
    y, u = L.fwd(save_u=True)
    assert api.marlaas_profile_read(L.ctx, api.MARLAAS_KERNEL_SHRINK)[1] == (0 if packed else 1)
    ref = oracle.fwd(w["x"], w["W"], w["A"], w["B"], w["ranks"], w["scales"], ids, layout=wl.TORCH)
    assert_close(to_host(y), ref, "y %d x %d" % (T, K))
