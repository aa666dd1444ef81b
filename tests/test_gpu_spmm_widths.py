"""The aggregation at every kind of width and row placement: widths that are no
multiple of 4 or 32, rows that start anywhere (odd strides and offsets), one
slice up to 256 columns and several past it, against the oracle (1e-5 S + 1e-7
per element), with the padding of X never used and that of Y never written.
Below F = 64 (where dense hub rows may take the column windows, another order,
on aligned rows) the result does not depend on how X and Y lie in memory: every
element is the same sum in the same order."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_11825_amd as agcn  # noqa: E402

from gpu_helpers import DEV, _dev, _mixed, _plan, assert_close  # noqa: E402


def _small(n=3000):
    rng = np.random.default_rng(4)
    return graphgen.random_csr(n, n, rng.integers(0, 29, size=n), seed=5)


@pytest.fixture(scope="module")
def graphs():
    return {"hubs": _mixed(71, n=6000, hub_max=4000), "small": _small(),
            "paper_params": _mixed(72, n=3000, hub_max=2000)}


def _place(X, offset, pad):
    """X with `pad` infinite columns after each row, `offset` floats past an aligned address."""
    n, F = X.shape
    buf = torch.full((n * (F + pad) + offset,), float("inf"), device=DEV)
    v = buf[offset:].view(n, F + pad)[:, :F]
    v.copy_(X)
    return v


@pytest.mark.parametrize("name", ["hubs", "small", "paper_params"])
@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 7, 9, 18, 31, 33, 35, 41, 61, 64, 65, 100, 127, 255,
                               257, 515])
def test_width_and_placement(graphs, name, F):
    g = graphs[name]
    kw = dict(max_block_waves=12, max_wave_nzs=32) if name == "paper_params" else {}
    plan = _plan(g, **kw)
    X = np.random.default_rng(F).standard_normal((g.n_cols, F)).astype(np.float32)
    Yr, S = oracle.spmm(g.rowptr, g.colidx, g.vals, X, n_cols=g.n_cols, want_scale=True)
    Xd = _dev(X)
    first = None
    for offset, pad in [(0, 0), (0, (-F) % 32), (1, 0), (2, 3), (32, 32 - F % 32 + 4)]:
        out = torch.full((g.n_rows * (F + pad) + offset,), 3.0, device=DEV)
        Yp = out[offset:].view(g.n_rows, F + pad)
        plan.spmm(_place(Xd, offset, pad), out=Yp[:, :F], act="relu")
        Y = Yp[:, :F].cpu().numpy()
        assert_close(Y, np.maximum(Yr, 0), S, f"{name} F={F} offset={offset} pad={pad}")
        assert torch.all(Yp[:, F:] == 3.0) and torch.all(out[:offset] == 3.0)
        if F < 64:
            first = Y if first is None else first
            assert np.array_equal(first.view(np.uint32), Y.view(np.uint32)), (F, offset, pad)
    plan.destroy()


@pytest.mark.parametrize("F", [33, 70])
def test_unaligned_workspace(graphs, F):
    """Hub-chunk partials in a workspace that starts 4 bytes past an aligned address."""
    g = graphs["hubs"]
    plan = _plan(g)
    X = _dev(np.random.default_rng(F).standard_normal((g.n_cols, F)).astype(np.float32))
    ws = torch.empty(plan.workspace_bytes(F) // 4 + 1, device=DEV)
    assert torch.equal(plan.spmm(X, ws=ws[1:]), plan.spmm(X))
    plan.destroy()


@pytest.mark.parametrize("n_rows,lo,hi", [(40000, 6, 10), (40000, 0, 60), (700, 6, 10)])
@pytest.mark.parametrize("F", [32, 64, 96, 128, 132])
def test_uniform_rows_over_many_columns(n_rows, lo, hi, F):
    """Rows of about one length over more columns than the L2s hold lines of
    (two-line slices on aligned rows), and of uneven length or few: the same
    bits as on rows that start anywhere."""
    rng = np.random.default_rng(n_rows + hi)
    g = graphgen.random_csr(n_rows, 270000, rng.integers(lo, hi + 1, size=n_rows), seed=hi, dupes=True)
    plan = _plan(g)
    X = np.random.default_rng(F).standard_normal((g.n_cols, F)).astype(np.float32)
    Yr, S = oracle.spmm(g.rowptr, g.colidx, g.vals, X, n_cols=g.n_cols, want_scale=True)
    Xd = _dev(X)
    Y = plan.spmm(Xd)
    assert_close(Y.cpu().numpy(), Yr, S, f"F={F}")
    assert torch.equal(Y, plan.spmm(_place(Xd, 1, 3)))
    plan.destroy()
