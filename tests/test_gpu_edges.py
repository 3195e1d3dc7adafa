"""Sizes at which a kernel's tiling or a rule of the dispatch changes, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_08527_amd import api

pytestmark = pytest.mark.gpu


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
