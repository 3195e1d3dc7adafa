"""One context on several streams, in branches of one graph and with many workspaces: calls that have a
workspace of their own do not meet in the context."""
import numpy as np
import pytest
import torch

from harness import workloads as wl
from helpers import HipLayer, assert_close, to_host
from paper_2605_08527_amd import api

pytestmark = pytest.mark.gpu

# few rows; some rows unsplit, split, with more workgroups than the chip holds beside the other's; the decode kernel
SIZES = [(12, 2048, 2048), (150, 1024, 2048), (70, 4200, 1024), (400, 1024, 4096)]


def _layers(seed, n=9):
    ctx = api.marlaas_create(0)
    out = []
    for i, (T, K, N) in enumerate(SIZES):
        rng = np.random.default_rng(seed + i)
        ids = rng.integers(-1, n, size=T).astype(np.int32)
        w = wl.make_layer(seed + i, T, K, N, [8 + 8 * (t % 3) for t in range(n)], [1.0] * n, ids, dtype="bf16", layout=wl.TORCH)
        out.append(HipLayer(w, ctx=ctx, table=True, packed=True))
    return ctx, out


def _alone(L):
    api.marlaas_set_workspace(L.ctx, L.ws)
    return L.fwd()[0]


def test_two_streams(oracle):
    ctx, layers = _layers(100)
    alone = [_alone(L) for L in layers]
    for L, y in zip(layers, alone):
        w = L.w
        assert_close(to_host(y), oracle.fwd(w["x"], w["W"], w["A"], w["B"], w["ranks"], w["scales"], w["ids"], layout=w["layout"]), "alone")
    streams = [torch.cuda.Stream() for _ in layers]
    for a in range(len(layers)):
        for b in range(a):
            ys = [[torch.empty_like(alone[i]) for _ in range(40)] for i in (a, b)]
            torch.cuda.synchronize()
            for k in range(40):
                for i, out in ((a, ys[0]), (b, ys[1])):
                    api.marlaas_set_workspace(ctx, layers[i].ws)
                    api.marlaas_lora_fwd(ctx, layers[i].desc, out[k], stream=streams[i])
            torch.cuda.synchronize()
            for i, out in ((a, ys[0]), (b, ys[1])):
                assert all(torch.equal(y, alone[i]) for y in out)


def test_branches_of_one_graph():
    ctx, layers = _layers(200)
    alone = [_alone(L) for L in layers]
    side = [torch.cuda.Stream() for _ in layers]
    ys = [torch.empty_like(y) for y in alone]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        main = torch.cuda.current_stream()
        for L, st, y in zip(layers, side, ys):
            st.wait_stream(main)
            api.marlaas_set_workspace(ctx, L.ws)
            api.marlaas_lora_fwd(ctx, L.desc, y, stream=st)
        for st in side:
            main.wait_stream(st)
    for rep in range(4):
        for y in ys:
            y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(y, a) for y, a in zip(ys, alone))
        assert torch.equal(_alone(layers[rep]), alone[rep])          # eager work between the replays


def test_workspace_first_seen_inside_a_capture():
    ctx, layers = _layers(300)
    L = layers[1]
    alone = _alone(L)
    ws = torch.empty_like(L.ws)
    y = torch.empty_like(alone)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.marlaas_set_workspace(ctx, ws)
        api.marlaas_lora_fwd(ctx, L.desc, y)
    for rep in range(3):
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, alone)
        assert torch.equal(_alone(L), alone)


def test_more_workspaces_than_areas():
    ctx, layers = _layers(400)
    alone = [_alone(L) for L in layers]
    keep = []
    for k in range(18):
        for L, y in zip(layers, alone):
            ws = torch.empty_like(L.ws)
            keep.append(ws)
            api.marlaas_set_workspace(ctx, ws)
            assert_close(to_host(L.fwd()[0]), to_host(y), "workspace %d" % k, tol_max=1e-3, tol_mean=2e-5)


def test_no_workspace_base_only_on_two_streams():
    rng = np.random.default_rng(5)
    ctx = api.marlaas_create(0)
    layers = []
    for T, K, N in SIZES:
        w = wl.make_layer(T, T, K, N, [], [], np.full(T, -1, dtype=np.int32), dtype="bf16", layout=wl.TORCH)
        L = HipLayer(w, ctx=ctx, packed=True)
        api.marlaas_set_workspace(ctx, None)
        layers.append(L)
    alone = [L.fwd()[0] for L in layers]
    streams = [torch.cuda.Stream() for _ in layers]
    ys = [[torch.empty_like(y) for _ in range(30)] for y in alone]
    torch.cuda.synchronize()
    for k in range(30):
        for L, st, out in zip(layers, streams, ys):
            api.marlaas_lora_fwd(ctx, L.desc, out[k], stream=st)
    torch.cuda.synchronize()
    for out, a in zip(ys, alone):
        assert all(torch.equal(y, a) for y in out)
