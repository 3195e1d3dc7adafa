"""Sizes at which a kernel's tiling or a rule of the dispatch changes, against the oracle."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from paper_2605_08527_amd import api
from test_gpu_parity import _check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    from oracle import lora_oracle
    return lora_oracle


# rows and columns around the 16-wide tiles, a contraction shorter than the waves' share, ranks around
# the 16-wide shrink tiles, more adapters in a row block than one pass takes, more than the inline table
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("T,K,N,ranks,table", [(1, 8, 8, [1], False), (5, 264, 40, [3, 17], True), (33, 512, 1032, [8, 16, 128], False),
                                               (48, 136, 520, [1 + 5 * (t % 7) for t in range(23)], False), (300, 1024, 1024, [16] * 4, True)])
def test_fp32_layer(oracle, T, K, N, ranks, table, layout):
    rng = np.random.default_rng(T)
    ids = rng.integers(-1, len(ranks), size=T).astype(np.int32)
    w = wl.make_layer(T, T, K, N, ranks, [0.5 + (t % 3) for t in range(len(ranks))], ids, dtype="f32", layout=layout, want_dY=True)
    _check_layer(oracle, w, bwd=True, tol=(1e-4, 1e-5), tag="fp32", table="table" if table else "lists")


@pytest.mark.parametrize("T,n", [(1, 1), (63, 800), (64, 1), (65, 2), (1024, 31), (1025, 32), (4097, 800), (4097, 801), (32768, 64), (32769, 64)])
def test_segment_map_one_launch_and_several(T, n):
    rng = np.random.default_rng(T * 7 + n)
    ctx = api.marlaas_create(0)
    m = api.marlaas_segmap_create(ctx, T, n)
    for batch in range(2):
        ids = rng.integers(-1, n, size=T).astype(np.int32)
        if batch:
            ids = np.sort(np.where(ids < 0, n, ids)).astype(np.int32)
            ids[ids == n] = -1
        api.marlaas_segmap_update(ctx, m, torch.from_numpy(ids).cuda(), n)
        perm, off = api.marlaas_segmap_export(m)
        key = np.where(ids < 0, n, ids)
        assert np.array_equal(perm, np.argsort(key, kind="stable"))
        assert np.array_equal(off, np.concatenate([[0], np.cumsum(np.bincount(key, minlength=n + 1))]))


# The large-batch GEMM: tile heights of 128, 192 and 256 rows with ragged last tiles, contractions that
# are no multiple of 64 (shorter than one k-tile, one and two k-tiles and a piece), the last round of
# tiles cut along the contraction, factors whose ranks leave the DMA path, more adapters in a row tile
# than a list of extra contraction tiles holds.
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("T,K,N,ranks,odd", [(4200, 40, 2056, [8, 16], False), (4200, 72, 2056, [8, 16], False), (4097, 136, 4104, [64, 8, 16, 128], False),
                                             (3070, 200, 4096, [16] * 5, True), (8300, 2048, 1032, [32, 8], False), (8300, 2048, 1032, [5, 24], True),
                                             (2500, 264, 8200, [128, 64] * 48, False)])
def test_large_batch_gemm_edges(oracle, T, K, N, ranks, odd, layout):
    rng = np.random.default_rng(T + K + N)
    ids = rng.integers(-1, len(ranks), size=T).astype(np.int32)
    if odd:
        ids = np.sort(ids)[::-1].copy()
    w = wl.make_layer(T + K, T, K, N, ranks, [0.5 + (t % 3) for t in range(len(ranks))], ids, dtype="bf16", layout=layout, want_dY=True)
    _check_layer(oracle, w, bwd=True, tag="wide")
    _check_layer(oracle, w, bwd=True, out_dtype=torch.bfloat16, tol=(1e-2, 2.5e-3), tag="wide bf16 out")


# Few rows on packed weights (one launch): row blocks of 16, 32 and 64, one to four column blocks per
# workgroup, contractions shorter than the waves' shares and no multiple of 32, ranks off the octets,
# adapters whose rows cross a row block, every row its own adapter, the bounded wait given up at once.
@pytest.mark.parametrize("spin", [None, "0"])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("T,K,N,ranks", [(1, 8, 8, [8]), (16, 1032, 264, [16] * 20), (17, 264, 6152, [128, 64, 8]), (32, 520, 12296, [24, 16]),
                                         (33, 2056, 1032, [8 + 8 * (t % 4) for t in range(40)]), (64, 4096, 4096, [16, 32]), (64, 296, 6160, [5, 13, 7])])
def test_few_rows_packed(oracle, monkeypatch, T, K, N, ranks, layout, spin):
    if spin is not None:
        monkeypatch.setenv("MARLAAS_SPIN_LIMIT", spin)
    rng = np.random.default_rng(T + K)
    ids = rng.integers(-1, len(ranks), size=T).astype(np.int32)
    if layout:
        ids = np.sort(ids)
    w = wl.make_layer(T + N, T, K, N, ranks, [0.5 + (t % 3) for t in range(len(ranks))], ids, dtype="bf16", layout=layout, want_dY=True)
    for rep in range(2):
        _check_layer(oracle, w, bwd=True, tag="few rows", table="table+packed")
    _check_layer(oracle, w, bwd=True, tag="few rows", table="lists+packed")


# Some more rows on packed weights, likewise in one launch: 64- and 80-row tiles of 64 and 128 columns, one,
# two and four contraction splits (fewer k-tiles in one than in the ring, none of them whole), more workgroups
# than the chip holds, more adapters than lanes, adapters across row tiles, ranks off the octets, the bounded
# waits given up at once.
@pytest.mark.parametrize("spin", [None, "0"])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("T,K,N,ranks", [(65, 136, 264, [8 + 8 * (t % 4) for t in range(70)]), (17, 9000, 520, [16, 8]), (80, 2056, 1032, [16] * 20),
                                         (160, 1032, 8200, [128, 8]), (157, 4104, 520, [24, 16]), (300, 1064, 3080, [5, 13, 7]),
                                         (385, 264, 1032, [16, 8, 64]), (1024, 136, 9000, [8] * 30)])
def test_some_rows_packed(oracle, monkeypatch, T, K, N, ranks, layout, spin):
    if spin is not None:
        if T * K > 200000:
            pytest.skip("the plain arithmetic after a wait given up takes long")
        monkeypatch.setenv("MARLAAS_SPIN_LIMIT", spin)
    rng = np.random.default_rng(T + K)
    ids = rng.integers(-1, len(ranks), size=T).astype(np.int32)
    if layout:
        ids = np.sort(ids)
    w = wl.make_layer(T + N, T, K, N, ranks, [0.5 + (t % 3) for t in range(len(ranks))], ids, dtype="bf16", layout=layout, want_dY=True)
    for rep in range(2):
        _check_layer(oracle, w, bwd=True, tag="some rows", table="table+packed")
    _check_layer(oracle, w, bwd=True, tag="some rows", table="lists+packed")
