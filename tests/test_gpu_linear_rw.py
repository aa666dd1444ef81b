"""k_linear_rw, the fp32 matrix instruction with W resident on chip: it serves
fin < 32 where fin, fout and the strides are multiples of 4, X, W and H 16-byte
aligned, and X and H under 4 GiB each. Whatever leaves those limits takes
k_linear_split and has to agree within both kernels' bound against 64 bits,
(fin + 12) u |X||W| (fin roundings here, fewer there)."""
import numpy as np
import pytest

import graphgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_11825_amd as agcn  # noqa: E402

from gpu_helpers import DEV, _dev, _mixed, _plan  # noqa: E402
from test_gpu_layer import _check_layer  # noqa: E402

U = 2.0 ** -24


def _xw(n, fin, fout, seed=0):
    gen = torch.Generator(device=DEV).manual_seed(n * 31 + fin * 7 + fout + seed)
    return (torch.randn((n, fin), generator=gen, device=DEV),
            torch.randn((fin, fout), generator=gen, device=DEV) / fin ** 0.5)


def _check(X, W, H):
    Xd, Wd = X.double(), W.double()
    err = (H.double() - Xd @ Wd).abs()
    assert (err <= (W.shape[0] + 12) * U * (Xd.abs() @ Wd.abs()) + 1e-30).all()


_LAST = {"one": lambda w: 1, "eighth": lambda w: w // 8, "eighth+1": lambda w: w // 8 + 1,
         "quarter+1": lambda w: w // 4 + 1, "half+1": lambda w: w // 2 + 1, "all-3": lambda w: w - 3}


@pytest.mark.parametrize("last", sorted(_LAST))
@pytest.mark.parametrize("fin,fout,short", [(4, 128, 3), (28, 128, 0), (12, 64, 5), (28, 60, 7), (16, 32, 1),
                                            (8, 8, 9)])
def test_last_round_split_by_columns(last, fin, fout, short):
    """The 16-row tiles of the last, partial round of resident waves are cut into
    1, 2, 4 or 8 column ranges. The grid is as many workgroups of 4 waves as are
    resident, 1 to 8 per CU by the kernel's registers, so every such count is
    tried. Rows of the last round are the same bits as inside a whole round."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for per_cu in range(1, 9):
        waves = cus * 4 * per_cu
        cut = 16 * waves
        n = cut + 16 * _LAST[last](waves) - short
        X, W = _xw(n, fin, fout)
        print(f"[rw tail] n={n} per_cu={per_cu} {last}", flush=True)
        H = agcn.linear(X, W)
        _check(X, W, H)
        Hr = agcn.linear(torch.cat([X[cut:], X[:cut]]).contiguous(), W)
        assert torch.equal(torch.cat([H[cut:], H[:cut]]), Hr)


@pytest.mark.parametrize("n,fin,fout,px,pw,ph,off", [
    (2051, 28, 44, 8, 4, 12, 0),        # padded rows, all 16-byte aligned
    (3001, 12, 128, 4, 8, 4, 0), (3001, 16, 260, 4, 4, 12, 0),   # three launches of 128 columns
    (3001, 28, 128, 0, 0, 3, 0), (3001, 28, 128, 0, 0, 0, 1),    # H's rows not 16-byte aligned
    (3001, 20, 64, 3, 0, 0, 0), (3001, 20, 64, 0, 1, 0, 0)])     # X's, W's
def test_padding_and_alignment(n, fin, fout, px, pw, ph, off):
    """Infinities in the padding of X and W are never used, the padding of H is
    never written, and each column is the same as in a launch of its own."""
    X, W = _xw(n, fin, fout)
    Xp = torch.full((n, fin + px), float("inf"), device=DEV)
    Wp = torch.full((fin, fout + pw), float("inf"), device=DEV)
    Xp[:, :fin], Wp[:, :fout] = X, W
    hb = torch.full((n * (fout + ph) + off,), 7.0, device=DEV)
    Hp = hb[off:].view(n, fout + ph)
    agcn.linear(Xp[:, :fin], Wp[:, :fout], out=Hp[:, :fout])
    _check(X, W, Hp[:, :fout])
    assert torch.all(Hp[:, fout:] == 7.0) and torch.all(hb[:off] == 7.0)
    if fout > 128:
        assert torch.equal(Hp[:, 128:256], agcn.linear(X, W[:, 128:256].contiguous()))


@pytest.mark.parametrize("big", ["X", "H"])
def test_spans_past_4_gib(big):
    """A span of 4 GiB or more is past the kernel's 32-bit offsets."""
    n, ld = 60_000, 18_000
    X, W = _xw(n, 28, 64)
    wide = torch.empty((n, ld), device=DEV)
    if big == "X":
        wide[:, :28] = X
        H = agcn.linear(wide[:, :28], W)
    else:
        H = wide[:, :64]
        agcn.linear(X, W, out=H)
    _check(X, W, H)


@pytest.mark.parametrize("fin,fout", [(16, 128), (28, 64), (4, 100), (12, 256), (20, 32), (24, 17)])
@pytest.mark.parametrize("act", ["relu", "none"])
def test_activation_in_the_layer(monkeypatch, fin, fout, act):
    """The layer's second order, (A X) W, ends in the linear kernel: its ReLU is
    applied at the writes of the whole rounds and of the last one."""
    monkeypatch.setenv("AGCN_HUB_WINDOWS", "0")
    g = _mixed(171, n=30000, hub_max=900)
    plan = _plan(g)
    X = np.random.default_rng(fin).standard_normal((g.n_cols, fin)).astype(np.float32)
    W = graphgen.weights(fin, fout, seed=fout)
    Y = _check_layer(plan, g, X, W, act)
    Z = agcn.linear(plan.spmm(_dev(X)), _dev(W))
    assert bool((Z < 0).any())
    if fout >= 100:     # (narrower: the first order)
        assert np.array_equal(Y, (Z.relu() if act == "relu" else Z).cpu().numpy())
    plan.destroy()
