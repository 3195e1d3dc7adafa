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
