"""agcn_gcn_layer's two orders, A (X W) and (A X) W: the layer aggregates first
where that gathers less (fin well below fout). Either way the layer's bound
against the oracle holds: (A X) W rounds the aggregation of |A||X| at 1e-5 and
the product at (fin + 12) u, both carried by S2 = |A||X||W|."""
import numpy as np
import pytest

import graphgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_11825_amd as agcn  # noqa: E402

from gpu_helpers import DEV, _dev, _mixed, _plan  # noqa: E402
from test_gpu_layer import _check_layer  # noqa: E402


@pytest.fixture(scope="module")
def graphs():
    return {"square": _mixed(161, n=7000, hub_max=900),
            "fewer_rows": _mixed(162, n=2500, n_cols=9000, hub_max=900),
            "more_rows": _mixed(163, n=9000, n_cols=2500, hub_max=900)}


# (The graphs' hub rows would take column windows, and such plans keep the first
# order: the second is reached without windows only.)
@pytest.mark.parametrize("windows", ["1", "0"])
@pytest.mark.parametrize("name", ["square", "fewer_rows", "more_rows"])
@pytest.mark.parametrize("fin,fout,pad", [(1, 64, 0), (3, 17, 0), (16, 33, 0), (32, 128, 0), (32, 40, 0),
                                          (30, 256, 3), (64, 65, 0), (100, 300, 0), (128, 256, 4)])
def test_layer_order_by_width(graphs, monkeypatch, name, fin, fout, pad, windows):
    monkeypatch.setenv("AGCN_HUB_WINDOWS", windows)
    g = graphs[name]
    plan = _plan(g)
    assert (plan.stats.hub_windows > 0) == (windows == "1")
    rng = np.random.default_rng(fin * 1000 + fout)
    X = rng.standard_normal((g.n_cols, fin)).astype(np.float32)
    W = graphgen.weights(fin, fout, seed=fout)
    Xp = torch.full((g.n_cols, fin + pad), float("nan"), device=DEV)
    Xp[:, :fin] = _dev(X)
    # exactly the workspace that the query asks for, followed by a guard
    nb = agcn.agcn_gcn_workspace_size(plan.handle, fout)
    buf = torch.full((nb // 4 + 64,), 6.0, device=DEV)
    for act in ("relu", "none"):
        Yp = torch.full((g.n_rows, fout + 4), 2.0, device=DEV)
        plan.gcn_layer(Xp[:, :fin], _dev(W), act=act, out=Yp[:, :fout], ws=buf)
        Y = Yp[:, :fout].cpu().numpy()
        _check_layer(plan, g, X, W, act, Yg=Y)
        assert torch.all(buf[nb // 4:] == 6.0) and torch.all(Yp[:, fout:] == 2.0)
        Y2 = plan.gcn_layer(_dev(X), _dev(W), act=act).cpu().numpy()
        if pad == 0:
            assert np.array_equal(Y.view(np.uint32), Y2.view(np.uint32))
        if windows == "0" and (fin, fout) in ((1, 64), (32, 128), (16, 33), (128, 256)):
            # whether the order is the one meant: the same kernels called one by one
            T = _dev(X) if name == "more_rows" else plan.spmm(_dev(X))
            Z = agcn.linear(T, _dev(W))
            Z = plan.spmm(Z, act=act) if name == "more_rows" else (Z.relu() if act == "relu" else Z)
            assert np.array_equal(Y2, Z.cpu().numpy())
    plan.destroy()


def test_layer_order_on_another_stream_and_captured(graphs, monkeypatch):
    monkeypatch.setenv("AGCN_HUB_WINDOWS", "0")
    g = graphs["square"]
    plan = _plan(g)
    assert plan.stats.hub_windows == 0 and int((g.degrees == 0).sum()) > 0
    W = _dev(graphgen.weights(32, 128, seed=5))
    X = torch.randn((g.n_cols, 32), device=DEV)
    Y0 = plan.gcn_layer(X, W)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    Y1 = torch.empty_like(Y0)
    ws = torch.empty(agcn.agcn_gcn_workspace_size(plan.handle, 128) // 4 + 1, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s), torch.cuda.graph(graph, stream=s):
        plan.gcn_layer(X, W, out=Y1, ws=ws, stream=s)
    for r in range(3):
        X.copy_(torch.randn_like(X))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y1, plan.gcn_layer(X, W)), f"replay {r}"
    del graph
    plan.destroy()


def test_layer_argument_errors_do_not_depend_on_the_order(graphs):
    g = graphs["square"]
    plan = _plan(g)
    X, W = torch.zeros((g.n_cols, 32), device=DEV), torch.zeros((32, 128), device=DEV)
    Y = torch.zeros((g.n_rows, 128), device=DEV)
    ws = torch.empty(agcn.agcn_gcn_workspace_size(plan.handle, 128) // 4 + 1, device=DEV)
    ok = [plan.handle, 32, 128, X.data_ptr(), 32, W.data_ptr(), 128, Y.data_ptr(), 128,
          ws.data_ptr(), None, 1]
    for at, value in [(3, None), (4, 31), (5, None), (6, 127), (7, None), (8, 127), (9, None),
                      (7, X.data_ptr()), (3, ws.data_ptr()), (11, 3)]:
        args = list(ok)
        args[at] = value
        with pytest.raises(agcn.AgcnError) as e:
            agcn.agcn_gcn_layer(*args)
        assert e.value.status == agcn.AGCN_ERR_INVALID_ARGUMENT
    plan.destroy()


@pytest.mark.parametrize("tiny", ["1", "0"])
@pytest.mark.parametrize("fin,fout", [(32, 128), (30, 256), (128, 32)])
def test_rows_without_nonzeros_are_zero_whatever_w_holds(graphs, monkeypatch, tiny, fin, fout):
    """A W that is not finite reaches every row with nonzeros and no other, in
    both orders, on two plan paths, on another stream and with a padded Y."""
    monkeypatch.setenv("AGCN_TEST_TINY", tiny)
    monkeypatch.setenv("AGCN_HUB_WINDOWS", "0")
    g = graphs["square"]
    plan = _plan(g)
    rng = np.random.default_rng(fin)
    X = _dev(rng.standard_normal((g.n_cols, fin)).astype(np.float32))
    W = graphgen.weights(fin, fout, seed=fout)
    W[3, :] = np.nan
    W = _dev(W)
    empty = _dev(g.degrees == 0)
    assert int(empty.sum()) > 100
    s = torch.cuda.Stream()
    for act in ("relu", "none"):
        Yp = torch.full((g.n_rows, fout + 3), 9.0, device=DEV)
        plan.gcn_layer(X, W, act=act, out=Yp[:, :fout])
        assert torch.all(Yp[empty, :fout] == 0) and torch.isnan(Yp[~empty, :fout]).all()
        assert torch.all(Yp[:, fout:] == 9.0)
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            Y = plan.gcn_layer(X, W, act=act)
        s.synchronize()
        assert torch.all(Y[empty] == 0) and torch.isnan(Y[~empty]).all()
    plan.destroy()


def test_empty_rows_of_larger_plans_are_zero():
    """The same through the short sort and through the multi-pass sort (a degree
    bound below the short sort's)."""
    deg = np.random.default_rng(7).integers(0, 9, size=60000)
    g = graphgen.random_csr(60000, 60000, deg, seed=8)
    empty = _dev(deg == 0)
    X, W = torch.randn((g.n_cols, 32), device=DEV), torch.full((32, 128), float("inf"), device=DEV)
    for kw in ({}, {"max_block_waves": 4, "max_wave_nzs": 32}):
        plan = _plan(g, **kw)
        Y = plan.gcn_layer(X, W, act="none")
        assert torch.all(Y[empty] == 0) and not torch.isfinite(Y[~empty]).any()
        plan.destroy()
