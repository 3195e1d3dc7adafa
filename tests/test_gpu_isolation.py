"""A tenant's adapter with infinities and NaN reaches that tenant's rows and gradients only, whatever
kernel serves the batch: rows of several adapters (and of none) share the 16-row blocks of the matrix
instructions, where a row takes the other adapters' factors times zero."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from helpers import HipLayer, assert_close, to_host

pytestmark = pytest.mark.gpu

# (T, K, N, ranks, dtype, packed weight, how decode calls are finished); the last two: large batches, whose
# shared row blocks are computed again in another order of sums
CASES = {
    "fp32": (70, 264, 1032, [8, 16, 40], "f32", False, None),
    "fp32 many": (640, 136, 2056, [16, 8, 8, 24], "f32", False, None),
    "few rows": (23, 520, 1032, [16, 8, 32], "bf16", True, None),
    "few rows, ranks off the octets": (30, 520, 1032, [12, 8, 20], "bf16", True, None),
    "some rows": (157, 1032, 1032, [16, 8, 64], "bf16", True, None),
    "some rows, split": (80, 4104, 520, [16] * 9, "bf16", True, None),
    "decode, second launch": (200, 1032, 1032, [16, 8, 64], "bf16", True, "2"),
    "decode, in the kernel": (200, 256, 1032, [16, 8, 64], "bf16", True, "1"),
    "decode, generic finish": (200, 1032, 1032, [16, 8, 64], "bf16", True, "0"),
    "small, not packed": (300, 1032, 520, [16, 8, 64], "bf16", False, None),
    "large": (4200, 264, 2056, [16, 8, 64], "bf16", False, None),
    "large, odd ranks, split last round": (2500, 1032, 4104, [5, 24, 128], "bf16", False, None),
}


def _poison(w, t):
    """The same workload, adapter t with a NaN and infinities in both factors."""
    bad = dict(w)
    nan, inf, ninf = (0x7fc0, 0x7f80, 0xff80) if w["dtype"] == "bf16" else (np.nan, np.inf, -np.inf)
    for k in ("A", "B"):
        bad[k] = [f.copy() for f in w[k]]
        flat = bad[k][t].reshape(-1)
        flat[0], flat[flat.size // 2], flat[-1] = nan, inf, ninf
    return bad


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_broken_adapter_stays_with_its_rows(monkeypatch, name, layout):
    T, K, N, ranks, dtype, packed, finish = CASES[name]
    if finish is not None:
        monkeypatch.setenv("MARLAAS_DECODE_FINISH", finish)
    rng = np.random.default_rng(T + K)
    n, t = len(ranks), 1
    ids = rng.integers(-1, n, size=T).astype(np.int32)
    w = wl.make_layer(T + N, T, K, N, ranks, [0.5 + (i % 3) for i in range(n)], ids, dtype=dtype, layout=layout, want_dY=True)
    out = []
    for v in (w, _poison(w, t)):
        L = HipLayer(v, want_bwd=True, packed=packed)
        y, u = L.fwd(save_u=True)
        out.append((y,) + L.bwd(u_saved=u))
    (y, dX, dA, dB), (yp, dXp, dAp, dBp) = out
    others = torch.from_numpy(ids != t).cuda()
    for a, b, what in ((y, yp, "y"), (dX, dXp, "dX")):
        assert not torch.isfinite(b[~others]).all(), what
        if name.startswith("large"):       # fp32 sums in another order, two-term split of u against fp32: 2^-17 of the term
            assert_close(to_host(b[others]), to_host(a[others]), what, tol_max=1e-4, tol_mean=1e-5)
        else:
            assert torch.equal(a[others], b[others]), what
    for i in range(n):
        if i != t:
            assert torch.equal(dA[i], dAp[i]) and torch.equal(dB[i], dBp[i])
