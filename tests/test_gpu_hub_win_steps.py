"""The window kernel's batches of every length: hub rows with 0 to 16 pairs and
far more per window -- spread, crowded into a few windows, repeated, gapped, in
the last (narrow) window only, one pair per window, and rows that ascend but
for one descent or not at all -- against the oracle, and the same bits twice."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import _dev, _plan, _spmm_check

torch = pytest.importorskip("torch")
import paper_2308_11825_amd as agcn  # noqa: E402

pytestmark = pytest.mark.gpu

N_COLS = 512 * 300 + 37         # two spans of 256 windows, the last window narrow


def _csr(rows):
    rowptr = np.zeros(len(rows) + 1, np.int64)
    rowptr[1:] = np.cumsum([r.size for r in rows])
    col = np.concatenate(rows).astype(np.int32)
    vals = np.random.default_rng(1).standard_normal(col.size).astype(np.float32)
    return graphgen.Graph("rows", len(rows), N_COLS, rowptr.astype(np.int32), col, vals)


def _spread(rng, d):
    return np.sort(rng.choice(N_COLS, size=d, replace=False))


def _rows():
    rng = np.random.default_rng(2)
    rows = [_spread(rng, int(d)) for d in rng.integers(9000, 16000, size=66)]
    rows += [np.sort(rng.integers(a, min(a + 1024, N_COLS), size=d)) for a, d in
             [(0, 20000), (512 * 255 + 7, 20000), (512 * 256 - 3, 32768), (700, 32769), (512 * 299, 40000)]]
    rows += [np.full(5000, 512 * 256), np.full(5000, 512 * 256 - 1), np.full(3000, N_COLS - 1),
             np.zeros(3000, np.int64), np.arange(0, N_COLS, 512), np.arange(511, N_COLS, 512)[:600]]
    rows[-2] = np.concatenate([rows[-2], [N_COLS - 1] * 400])
    for at in [1, 3, 4, 255, 256, 257, 2047, 2048, 2049, 8000, 9999]:
        r = _spread(rng, 10000)
        r[at - 1], r[at] = r[at], r[at - 1]      # one descent, before element `at`
        rows.append(r)
    rows.append(_spread(rng, 12000)[::-1])
    r = _spread(rng, 12000)
    rows.append(np.concatenate([r[6000:], r[:6000]]))
    rows += [_spread(rng, d) for d in range(600, 5400, 300)]   # 2 to 18 per window
    rng.shuffle(rows)
    small = [np.sort(rng.choice(N_COLS, size=int(d), replace=False)) for d in
             rng.integers(0, 9, size=500)]
    return rows + small


@pytest.mark.parametrize("F", [64, 100])
def test_window_batches(F):
    g = _csr(_rows())
    p = _plan(g)
    assert p.stats.hub_windows == 301
    Y = _spmm_check(p, g, F, seed=F)
    X = np.random.default_rng(F).standard_normal((g.n_cols, F)).astype(np.float32)
    assert np.array_equal(p.spmm(_dev(X)).cpu().numpy().view(np.uint32), Y.view(np.uint32))
    p.destroy()


@pytest.mark.parametrize("F", [64, 132])
def test_masked_pairs_never_meet_x(F):
    """X rows that open a window hold infinities and NaN. Hub rows that reference
    none of them stay finite, whatever the lengths of their last batches and of
    their neighbours', and whether or not their columns ascend; all rows match the
    oracle, which multiplies stored pairs only."""
    rows = [r[r % 512 != 0] if k % 3 else r for k, r in enumerate(_rows())]
    g = _csr(rows)
    p = _plan(g)
    assert p.stats.hub_windows == 301
    X = np.random.default_rng(F).standard_normal((g.n_cols, F)).astype(np.float32)
    X[0::1024], X[512::1024] = np.inf, np.nan
    Y = _spmm_check(p, g, F, X=X)
    free = np.array([k for k, r in enumerate(rows) if not (r % 512 == 0).any()])
    assert free.size > 50 and np.isfinite(Y[free]).all()
    p.destroy()
