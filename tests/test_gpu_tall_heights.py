"""Some rows in tall tiles, each where the planner takes it and with u laid over the sums where its height can have it; that the planner takes what
a name says is checked by tests/test_tall_heights.py."""
import numpy as np
import pytest
import torch

import test_gpu_tall_tiles as tall
from helpers import HipLayer

pytestmark = pytest.mark.gpu

# (rows, contraction, columns, ranks); the number of the name is the tile that the planner takes.  u lies over the sums in tiles of 256 rows
# from rank 32 on, of 160 from 112, of 96 above 64.
CASES = {
    "96, whole tiles": (288, 2056, 10240, [16] * 4), "96, u over the sums": (288, 2056, 10240, [128] * 4),
    "96, u over the sums, last tile short": (512, 5120, 5120, [128] * 8),
    "96, jobs whole, two pieces are more than fit": (512, 5120, 5120, [32] * 64), "96, the same with a tile of one row": (481, 3080, 5120, [32] * 60),
    "128": (128, 4104, 28664, [16] * 32), "128, rank 128": (128, 4096, 28672, [128] * 4),
    "160": (157, 3208, 28672, [16] * 70), "160, several jobs each": (320, 3208, 14336, [16, 8] * 20), "160, few with rows": (160, 3208, 28672, [16] * 32),
    "160, u over the sums, last tile short": (310, 5128, 14336, [128] * 4), "160, u over the sums, last tile whole": (320, 5128, 14336, [112] * 4),
    "256": (256, 3080, 28672, [16, 8] * 16), "256, u over the sums": (512, 4096, 14336, [32] * 32),
    "256, u over the sums, last tile short": (250, 4104, 28672, [64] * 8), "256, u over the sums, rank 128": (256, 4104, 28672, [128, 100] * 2),
}


@pytest.mark.parametrize("spin", [None, "0"])
@pytest.mark.parametrize("name", list(CASES))
def test_tall_heights(oracle, monkeypatch, name, spin):
    monkeypatch.setitem(tall.CASES, name, CASES[name])
    tall.test_tall_tiles(oracle, monkeypatch, name, spin)


# (in tiles of 96, 128, 160 and 256 rows)
WITHOUT = [(512, 3080, 5120), (97, 4096, 28672), (320, 3208, 14336), (255, 3080, 28672)]


@pytest.mark.parametrize("T,K,N", WITHOUT)
def test_without_adapters(oracle, T, K, N):
    tall.test_without_adapters(oracle, T, K, N)


def test_broken_adapter_stays_with_its_rows():
    T, K, N, ranks = 157, 3208, 28672, [16] * 32
    w = tall._layer(T, K, N, ranks, seed=2)
    bad = dict(w)
    for k in ("A", "B"):
        bad[k] = [f.copy() for f in w[k]]
        flat = bad[k][1].reshape(-1)
        flat[0], flat[flat.size // 2], flat[-1] = 0x7fc0, 0x7f80, 0xff80
    y, yb = (HipLayer(v, table=True, packed=True).fwd()[0] for v in (w, bad))
    others = torch.from_numpy(w["ids"] != 1).cuda()
    assert torch.equal(y[others], yb[others]) and not torch.isfinite(yb[~others]).all()
