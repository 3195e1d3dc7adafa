"""The grouping of one launch against numpy's stable sort, where its waves' shares begin and end: 64 tokens a wave and
step, 256 that stay in registers (4096 in the block), a wave of buckets, the largest batch it takes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 800])
@pytest.mark.parametrize("T", [1, 64, 65, 1023, 1025, 4096, 4097, 32768])
def test_grouping(T, n):
    from paper_2605_08527_amd import api
    rng = np.random.default_rng(1000 * n + T)
    ids = rng.integers(-1, n, size=T).astype(np.int32)
    ctx = api.marlaas_create(0)
    m = api.marlaas_segmap_create(ctx, T, n)
    for batch in (ids, np.sort(ids)[::-1].copy(), np.full(T, n - 1, dtype=np.int32), ids):
        api.marlaas_segmap_update(ctx, m, torch.from_numpy(batch).cuda(), n)
        perm, seg_off = api.marlaas_segmap_export(m)
        bucket = np.where(batch < 0, n, batch)
        assert np.array_equal(perm, np.argsort(bucket, kind="stable"))
        assert np.array_equal(seg_off, np.concatenate([[0], np.cumsum(np.bincount(bucket, minlength=n + 1))]))
    with pytest.raises(api.MarlaasError):
        api.marlaas_segmap_update(ctx, m, torch.full((T,), n, dtype=torch.int32, device="cuda"), n)
