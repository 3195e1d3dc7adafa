"""Launches on one workspace take turns over two areas for u, each clearing what the one before it left, and leave the area of
the partial sums alone after somebody gave up waiting.  Calls with more, fewer and no adapters' values to exchange, with
and without contraction splits, in turn on one context: every call has the bits of the same call on a context of its own."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from helpers import HipLayer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spin", [None, "0", "1", "3"])
def test_calls_take_turns(monkeypatch, spin):
    if spin is not None:
        monkeypatch.setenv("MARLAAS_SPIN_LIMIT", spin)
    layers, alone = [], []
    # split contraction, most of u; no split; split without adapters; few rows (an area of their own); split again; fewer
    # workgroups than there are lines to count them
    for T, K, N, ranks in [(157, 4104, 520, [64, 128]), (300, 1064, 3080, [8] * 40), (100, 4104, 1032, None), (17, 264, 1032, [16]), (80, 4104, 264, [16] * 30),
                           (65, 264, 72, [16])]:
        rng = np.random.default_rng(T + K)
        ids = np.full(T, -1, dtype=np.int32) if ranks is None else rng.integers(-1, len(ranks), size=T).astype(np.int32)
        ranks = ranks or [8]
        w = wl.make_layer(T + N, T, K, N, ranks, [0.5 + t % 3 for t in range(len(ranks))], ids, dtype="bf16", layout=wl.TORCH)
        L = HipLayer(w, table=True, packed=True)
        alone.append(L.fwd()[0].clone())
        layers.append(L)
    ctx = layers[0].ctx
    ws = torch.empty(max(L.ws.numel() for L in layers if L.ws is not None), dtype=torch.uint8, device="cuda")
    from paper_2605_08527_amd import api
    api.marlaas_set_workspace(ctx, ws)
    for rnd in range(3):
        for i in range(len(layers)):
            k = (i * (rnd + 1)) % len(layers) if rnd < 2 else i
            L = layers[k]
            y = torch.full_like(alone[k], 7.0)
            api.marlaas_lora_fwd(ctx, L.desc, y)
            if rnd == 1:
                api.marlaas_lora_fwd(ctx, L.desc, y)
            assert torch.equal(y, alone[k]), (rnd, k)


def test_most_values_to_exchange(oracle):
    """Eight projections of 1024 rows and ranks of 128, a contraction whose u is computed in two pieces: an area of u is full
    to its end.  Calls in turn, the areas and their clearing as well."""
    from paper_2605_08527_amd import api
    from helpers import assert_close, to_dev, to_host
    T, K, N, n, P = 1024, 6408, 72, 3, 8
    ids = np.random.default_rng(2).integers(-1, n, size=T).astype(np.int32)
    ws = [wl.make_layer(300 + p, T, K, N, [128, 128, 120], [0.5, 1.0, 2.0], ids, dtype="bf16", layout=wl.TORCH) for p in range(P)]
    ctx = api.marlaas_create(0)
    seg = api.marlaas_segmap_build(ctx, torch.from_numpy(ids).cuda(), n)
    x = to_dev(ws[0]["x"])
    table = api.marlaas_adapter_table_create(ctx, n, P, 128)
    keep, descs, ys = [], [], []
    for p, w in enumerate(ws):
        W, A, B = to_dev(w["W"]), [to_dev(a) for a in w["A"]], [to_dev(b) for b in w["B"]]
        for t in range(n):
            api.marlaas_adapter_table_update(ctx, table, p, t, A[t], B[t], w["ranks"][t], w["scales"][t])
        packed = api.marlaas_pack_weight(ctx, W, api.MARLAAS_LAYOUT_TORCH, 0)
        keep.append((A, B, packed))
        descs.append(api.LoraDesc(x, W, None, None, w["ranks"], w["scales"], seg, layout=wl.TORCH, out_dtype=torch.float32, table=table, proj=p, W_packed_fwd=packed))
        ys.append(torch.empty((T, N), dtype=torch.float32, device="cuda"))
    buf = torch.empty(max(api.marlaas_workspace_bytes_multi(descs), 256), dtype=torch.uint8, device="cuda")
    api.marlaas_set_workspace(ctx, buf)
    api.marlaas_profile_enable(ctx, True)
    api.marlaas_lora_fwd_multi(ctx, descs, ys)
    torch.cuda.synchronize()
    assert api.marlaas_profile_read(ctx, api.MARLAAS_KERNEL_GEMM)[1] == 1
    api.marlaas_profile_enable(ctx, False)
    for p, (w, y) in enumerate(zip(ws, ys)):
        ref = oracle.fwd(ws[0]["x"], w["W"], w["A"], w["B"], w["ranks"], w["scales"], ids, layout=wl.TORCH)
        assert_close(to_host(y), ref, "projection %d" % p, 1e-2, 1e-3)
    first = [y.clone() for y in ys]
    for rnd in range(4):
        k = 2 if rnd % 2 else P
        api.marlaas_lora_fwd_multi(ctx, descs[:k], ys[:k])
        for y, f in zip(ys, first):
            if rnd % 2 == 0:
                assert torch.equal(y, f), rnd
