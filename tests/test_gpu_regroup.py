"""A captured forward of few rows on packed weights serves the batches that its segment map is given later:
the kernels take the grouping from the map when they run, not from the capture."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from helpers import HipLayer, assert_close, to_host
from paper_2605_08527_amd import api

pytestmark = pytest.mark.gpu


def _groupings(rng, T, n):
    one = np.zeros(T, dtype=np.int32)                        # grouped already, a single adapter
    base = np.where(rng.random(T) < 0.9, -1, rng.integers(0, n, size=T)).astype(np.int32)
    base[0] = n - 1
    return [one, rng.integers(0, n, size=T).astype(np.int32), (np.arange(T) % n).astype(np.int32), base,
            np.sort(rng.integers(0, n, size=T)).astype(np.int32), np.full(T, n - 1, dtype=np.int32)]


# few rows and some more; adapters up to the lanes of a wave and above, ranks of one to eight 16-wide tiles,
# tiles of 64 and 80 rows, a split contraction; captured with one adapter and with all of them
@pytest.mark.parametrize("T,K,N,ranks", [(23, 520, 1032, [16, 8, 40]), (60, 1032, 520, [8 + 8 * (t % 16) for t in range(70)]), (60, 4200, 1024, [16] * 9),
                                         (157, 1032, 4104, [16] * 32), (300, 264, 8200, [8, 16, 32, 64] * 16), (384, 136, 1032, [128] * 130)])
@pytest.mark.parametrize("first", [0, 2])
def test_replay_after_regroup(oracle, T, K, N, ranks, first):
    n = len(ranks)
    rng = np.random.default_rng(T + n)
    maps = _groupings(rng, T, n)
    maps = maps[first:] + maps[:first]
    w = wl.make_layer(T + N, T, K, N, ranks, [0.5 + t % 3 for t in range(n)], maps[0], dtype="bf16", layout=wl.TORCH)
    L = HipLayer(w, table=True, packed=True)
    y = torch.empty((T, N), dtype=torch.float32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.marlaas_lora_fwd(L.ctx, L.desc, y)
    for ids in maps:
        api.marlaas_segmap_update(L.ctx, L.map, torch.from_numpy(ids).cuda(), n)
        ref = oracle.fwd(w["x"], w["W"], w["A"], w["B"], w["ranks"], w["scales"], ids, layout=wl.TORCH)
        for rep in range(3):
            y.fill_(float("nan"))
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            assert_close(to_host(y), ref, "replay")
            assert beg.elapsed_time(end) < 50.0              # (a wait given up costs as many milliseconds and more)
        eager, _ = L.fwd()                                   # the program's own work between the replays
        assert torch.equal(eager, y) or np.allclose(to_host(eager), to_host(y), rtol=1e-4, atol=1e-4)


# A pass of many rows is captured again after an update; where it is not, and the map has fewer rows with adapters
# than it had, the shrink whose contraction is split writes none of the rows that have no adapter any more.
@pytest.mark.parametrize("layout", [0, 1])
def test_split_shrink_replayed_with_fewer_rows(layout):
    T, K, N, n = 4200, 264, 4104, 40
    rng = np.random.default_rng(layout)
    ids = rng.integers(0, n, size=T).astype(np.int32)
    w = wl.make_layer(T, T, K, N, [8 + 8 * (t % 4) for t in range(n)], [1.0] * n, ids, dtype="bf16", layout=layout)
    L = HipLayer(w, table=True)
    y = torch.empty((T, N), dtype=torch.float32, device="cuda")
    u = torch.empty((T, api.marlaas_u_stride(L.desc)), dtype=torch.float32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.marlaas_lora_fwd(L.ctx, L.desc, y, u_save=u)
    for rows in (4200, 3997, 64, 1):
        ids[rng.permutation(T)[:T - rows]] = -1
        left = int((ids >= 0).sum())
        api.marlaas_segmap_update(L.ctx, L.map, torch.from_numpy(ids).cuda(), n)
        u.fill_(7.0)
        graph.replay()
        got = u.clone()
        u.fill_(7.0)
        api.marlaas_lora_fwd(L.ctx, L.desc, y, u_save=u)
        torch.cuda.synchronize()
        assert bool((got[left:] == 7.0).all())
        assert_close(to_host(got[:left]), to_host(u[:left]), "u of the rows left", tol_max=1e-3, tol_mean=2e-5)
