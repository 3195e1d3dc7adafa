"""Some rows in tall tiles (96, 128, 160 and 256 rows): edges of tiles, contractions that end inside a k-tile or a ring, more adapters than lanes,
ranks off the octets, producers with several jobs each and with none, and waits given up at once."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from helpers import HipLayer, assert_close, to_host

pytestmark = pytest.mark.gpu


def _layer(T, K, N, ranks, seed=0, share=None):
    rng = np.random.default_rng(T + K + seed)
    ids = rng.integers(-1, len(ranks), size=T).astype(np.int32)
    if share is not None:                                        # (few adapters with rows: most producers' jobs do not exist)
        ids = np.where(ids < share, ids, -1).astype(np.int32)
    return wl.make_layer(T + N, T, K, N, ranks, [0.5 + t % 3 for t in range(len(ranks))], ids, dtype="bf16", layout=wl.TORCH)


# (rows, contraction, columns, ranks)
CASES = {
    "96, last tile of one row": (481, 3080, 5120, [8, 16, 32, 64] * 8), "96, whole tiles": (288, 2056, 10240, [16] * 4), "96, ranks off the octets": (257, 2120, 10232, [16, 12, 20]),
    "128": (128, 2056, 28664, [16] * 32), "128, last tile short": (200, 3000, 14336, [32] * 40),
    "160": (157, 2056, 28672, [16] * 70), "160, several jobs each": (320, 2056, 14336, [16, 8] * 20), "160, few with rows": (160, 2056, 28672, [16] * 32),
    "256": (256, 2056, 28672, [16, 8] * 16), "256, last tile short": (490, 4104, 14344, [16] * 8),
}


@pytest.mark.parametrize("spin", [None, "0"])
@pytest.mark.parametrize("name", list(CASES))
def test_tall_tiles(oracle, monkeypatch, name, spin):
    if spin is not None:
        monkeypatch.setenv("MARLAAS_SPIN_LIMIT", spin)
    T, K, N, ranks = CASES[name]
    w = _layer(T, K, N, ranks, share=2 if "few" in name else None)
    L = HipLayer(w, table=True, packed=True)
    y, u = L.fwd(save_u=True)
    ys = [L.fwd()[0] for _ in range(2)]                          # (both areas of u, each cleared by the launch after)
    assert all(torch.equal(y, v) for v in ys)
    cols = np.r_[0:160, N // 2 - 70:N // 2 + 70, N - 136:N]
    ref = oracle.fwd(w["x"], np.ascontiguousarray(w["W"][cols]), w["A"], [np.ascontiguousarray(b[cols]) for b in w["B"]], w["ranks"], w["scales"], w["ids"], layout=wl.TORCH)
    assert_close(to_host(y)[:, cols], ref, name)
    other = "MARLAAS_DECODE_FINISH"                              # all columns against the split kernel with its own launch
    monkeypatch.setenv(other, "2")
    z, _ = HipLayer(w, table=True, packed=True).fwd()
    assert_close(to_host(y), to_host(z), name + ", all columns", tol_max=1e-4, tol_mean=1e-5)


@pytest.mark.parametrize("T,K,N", [(512, 1160, 6144), (97, 4096, 28672), (320, 2304, 14336), (255, 2304, 28672)])
def test_without_adapters(oracle, T, K, N):
    w = _layer(T, K, N, [8], seed=1)
    w["ids"] = np.full(T, -1, dtype=np.int32)
    y, _ = HipLayer(w, table=True, packed=True).fwd()
    cols = np.r_[0:136, N - 136:N]
    assert_close(to_host(y)[:, cols], wl_product(w, cols), "%d rows" % T)


def wl_product(w, cols):
    f = lambda a: wl.bf16_bits_to_f32(a).astype(np.float64)
    return f(w["x"]) @ f(np.ascontiguousarray(w["W"][cols])).T


def test_broken_adapter_stays_with_its_rows():
    T, K, N, ranks = 157, 2056, 28672, [16] * 32
    w = _layer(T, K, N, ranks, seed=2)
    bad = dict(w)
    for k in ("A", "B"):
        bad[k] = [f.copy() for f in w[k]]
        flat = bad[k][1].reshape(-1)
        flat[0], flat[flat.size // 2], flat[-1] = 0x7fc0, 0x7f80, 0xff80
    y, yb = (HipLayer(v, table=True, packed=True).fwd()[0] for v in (w, bad))
    others = torch.from_numpy(w["ids"] != 1).cuda()
    assert torch.equal(y[others], yb[others]) and not torch.isfinite(yb[~others]).all()
