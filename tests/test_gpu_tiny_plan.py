"""The single-workgroup plan (at most 16384 rows and 2^18 - 1 nonzeros) at its
edges: rows per thread (multiples of 1024), digits of the degree sort (5 bits),
the largest degree that its packed rows hold, no nonzeros at all, a column
index out of range at every place of the last 16-byte group, and index arrays
that start 4 bytes past an aligned address. The plan equals the oracle's bit
for bit, also past the limits, where the other paths run."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import _dev, _plan, _spmm_check, assert_plan_matches_oracle

torch = pytest.importorskip("torch")
import paper_2308_11825_amd as agcn  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(g, **kw):
    p = _plan(g, **kw)
    assert_plan_matches_oracle(p, g)
    _spmm_check(p, g, 5)
    p.destroy()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 1023, 1024, 1025, 2048, 3000, 16383, 16384, 16385])
def test_rows(n):
    rng = np.random.default_rng(n)
    _check(graphgen.random_csr(n, 500, rng.integers(0, 16, size=n), seed=n))


@pytest.mark.parametrize("degrees", [[0], [1], [31], [32], [0, 31, 32, 33], [1023], [1024, 5], [7, 32767],
                                     [0, 0, 32768], [131072], [200000, 31]])
def test_degree_digits(degrees):
    """Stable order among equal degrees, in one to four passes (or none)."""
    rng = np.random.default_rng(len(degrees))
    deg = rng.choice(np.minimum(degrees, 40), size=3000)
    deg[[17, 2999]] = max(degrees)
    deg[:17] = degrees[0] if degrees[0] < 200 else 2
    g = graphgen.random_csr(3000, 2000, deg, seed=7, dupes=True)
    _check(g)
    _check(g, max_block_waves=32, max_wave_nzs=64)
    _check(g, max_block_waves=1, max_wave_nzs=1)


@pytest.mark.parametrize("nnz", [(1 << 18) - 1, 1 << 18])
def test_most_nonzeros(nnz):
    deg = np.full(4, nnz // 4)
    deg[:nnz % 4] += 1
    _check(graphgen.random_csr(4, 1000, deg, seed=9, dupes=True))
    deg = np.array([0, nnz, 0])           # one row holds every nonzero
    _check(graphgen.random_csr(3, 1000, deg, seed=10, dupes=True))


@pytest.mark.parametrize("nnz", [5, 4096, 65536 + 3, 131072 + 1])
def test_bad_column_anywhere(nnz):
    n = 300
    deg = np.full(n, nnz // n)
    deg[:nnz % n] += 1
    g = graphgen.random_csr(n, 77, deg, seed=11, dupes=True)
    at = {0, 1, nnz // 2, nnz - 1, nnz - 2, nnz - 3, nnz - 4, nnz - 5} | set(range(60000, nnz, 8191))
    for k in sorted(at):
        for bad in (77, -1):
            col = g.colidx.copy()
            col[k] = bad
            with pytest.raises(agcn.AgcnError) as e:
                agcn.Plan(_dev(g.rowptr), _dev(col), _dev(g.vals), n_cols=77)
            assert e.value.status == agcn.AGCN_ERR_INVALID_INPUT and "column" in str(e.value)
    _check(g)


def test_unaligned_index_arrays():
    rng = np.random.default_rng(3)
    g = graphgen.random_csr(5000, 4000, rng.integers(0, 40, size=5000), seed=12)
    off = lambda a: torch.cat([torch.zeros(1, dtype=_dev(a).dtype, device="cuda:0"), _dev(a)])[1:]
    p = agcn.Plan(off(g.rowptr), off(g.colidx), off(g.vals), n_cols=4000)
    assert_plan_matches_oracle(p, g)
    p.destroy()
