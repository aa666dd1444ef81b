"""agcn_linear's kernels at the sizes where they can go wrong: chunks of 32 k
(edges and remainders), tiles of 16 to 256 columns and 16 to 128 rows, the
k split for few rows, unaligned data, and values outside bf16's range.

Tolerance per element: (fin + 12) u |X||W| + 8 fin 2^-149 (u = 2^-24). The parts'
products are exact; an element sees ceil(fin / 32) matrix instructions and as
many fp32 adds on its leading products, off by at most 2 u and 1 u of the
largest partial sum (at most |X||W|), which is at most fin + 3 u for every fin
here; the sums of the small products are below 2^-6 |X||W| and their errors
below 1 u, the products left out below 2^-34; bits lost below bf16's smallest
number are at most 2^-26 of an element that is kept. Each of the eight products
of a term is off by at most 2^-149 where it is subnormal.
"""
import numpy as np
import pytest

import graphgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_11825_amd as agcn  # noqa: E402

from gpu_helpers import DEV, _dev  # noqa: E402

U = 2.0 ** -24


def _check(X, W, H):
    fin = W.shape[0]
    with np.errstate(invalid="ignore", over="ignore"):
        ref = X.astype(np.float64) @ W.astype(np.float64)
        S = np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64))
        ref32 = ref.astype(np.float32)
        finite = np.isfinite(ref32)
        assert np.array_equal(np.isnan(H), np.isnan(ref32))
        assert np.array_equal(H[~finite & ~np.isnan(ref32)], ref32[~finite & ~np.isnan(ref32)])
        err = np.abs(H.astype(np.float64) - ref)[finite]
    tol = ((fin + 12) * U * S + 8 * fin * 2.0 ** -149)[finite]
    assert (err <= tol).all(), (float((err / tol).max()), X.shape, W.shape)


def _xw(n, fin, fout):
    rng = np.random.default_rng(n * 7 + fin * 3 + fout)
    return rng.standard_normal((n, fin)).astype(np.float32), graphgen.weights(fin, fout, seed=n + fout)


# rows: one, a remainder of every row tile, past the k split's line; fin: chunk
# edges; fout: edges of every column tile (16, 32, 48, 64, 128, 256)
@pytest.mark.parametrize("n,fin,fout", [
    (1, 1, 1), (15, 31, 15), (17, 33, 17), (16, 64, 16), (129, 65, 33), (63, 256, 48), (65, 257, 49),
    (3000, 1000, 16), (1000, 300, 130), (3001, 95, 64), (20000, 36, 65), (40001, 32, 47),
    (40003, 29, 48), (66000, 64, 64), (70000, 66, 128), (70001, 100, 129), (40000, 256, 255),
    (33000, 259, 256), (70000, 31, 3), (40007, 127, 1), (50000, 12, 132), (100003, 28, 32)])
def test_linear_tile_edges(n, fin, fout):
    X, W = _xw(n, fin, fout)
    print(f"[linear split] n={n} fin={fin} fout={fout}", flush=True)
    _check(X, W, agcn.linear(_dev(X), _dev(W)).cpu().numpy())


@pytest.mark.parametrize("n,fin,fout", [(2049, 70, 41), (70000, 70, 41), (40000, 300, 200)])
def test_linear_unaligned_rows_and_padding(n, fin, fout):
    """Odd offsets and strides on every matrix; infinities in the padding of X
    and W are never used, the padding of H never written."""
    X, W = _xw(n, fin, fout)
    xb = torch.full((n * (fin + 3) + 1,), float("inf"), device=DEV)
    Xd = xb[1:].view(n, fin + 3)[:, :fin]
    Xd.copy_(_dev(X))
    wb = torch.full((fin * (fout + 1) + 3,), float("nan"), device=DEV)
    Wd = wb[3:].view(fin, fout + 1)[:, :fout]
    Wd.copy_(_dev(W))
    hb = torch.full((n * (fout + 5) + 2,), 4.0, device=DEV)
    Hp = hb[2:].view(n, fout + 5)
    agcn.linear(Xd, Wd, out=Hp[:, :fout])
    _check(X, W, Hp[:, :fout].cpu().numpy())
    assert torch.all(Hp[:, fout:] == 4.0) and torch.all(hb[:2] == 4.0)


@pytest.mark.parametrize("n", [500, 40000])     # the k split, the tiles
def test_linear_infinities_nan_and_extreme_values(n):
    """Elements that meet an infinity or a NaN, or values that round past
    bf16's largest, come out as in a float32 product; their neighbours are not
    touched. Zero times infinity is NaN, an infinity times a weight infinite."""
    X, W = _xw(n, 70, 40)
    X[3, 5], X[4, 69], X[5, 0], X[6, 33] = np.inf, -np.inf, np.nan, 3.4e38
    X[7], X[8], X[9] = 0.0, 1e-39, 1e-42
    X[n - 1, 1] = np.inf
    W[5, 3], W[69, 7] = 0.0, -2.0
    W[10, 11] = np.inf
    W[33, :] = 0.25
    H = agcn.linear(_dev(X), _dev(W)).cpu().numpy()
    _check(X, W, H)
    assert np.isnan(H[3, 3]) and np.isinf(H[4, 7]) and np.isfinite(H[6, :11]).all()
    clean = agcn.linear(_dev(X[20:21]), _dev(W)).cpu().numpy()
    assert np.isfinite(np.delete(H[20], 11)).all() and np.isfinite(np.delete(clean[0], 11)).all()


def _chain(X, W):
    """One fp32 rounding per term, in order: what a fused multiply-add makes
    (a product of two floats is exact in double)."""
    H = np.zeros((X.shape[0], W.shape[1]), np.float32)
    for k in range(X.shape[1]):
        H = (H.astype(np.float64) + X[:, k:k + 1].astype(np.float64) * W[k].astype(np.float64)).astype(np.float32)
    return H


@pytest.mark.parametrize("n", [600, 20000])     # the k split, the tiles
@pytest.mark.parametrize("fin,nz", [(128, 1), (128, 2), (128, 3), (128, 8), (300, 4), (1, 1), (2, 2), (3, 3),
                                    (33, 33), (256, 256)])
def test_linear_error_is_at_most_one_rounding_per_term(n, fin, nz):
    """Rows of few nonzeros, spread over the chunks, and dense ones: the 2-norm
    error against 64 bits is at most that of a chain of fused multiply-adds
    (1.02: the spread of a sample), and an element that is one product is off by
    at most u for its one rounding plus u / 8 for the seven small sums (each at
    most 2^-7 of it and off by 2^-23 of itself)."""
    rng = np.random.default_rng(n + fin + nz)
    W = rng.standard_normal((fin, 40)).astype(np.float32)
    X = np.zeros((n, fin), np.float32)
    at = np.argsort(rng.random((n, fin)), axis=1)[:, :nz]
    np.put_along_axis(X, at, rng.standard_normal((n, nz)).astype(np.float32), axis=1)
    H = agcn.linear(_dev(X), _dev(W)).cpu().numpy()
    ref = X.astype(np.float64) @ W.astype(np.float64)
    err = np.abs(H - ref)
    chain = np.linalg.norm(_chain(X, W) - ref)
    assert np.linalg.norm(err) <= 1.02 * chain, (np.linalg.norm(err) / np.linalg.norm(ref),
                                                 chain / np.linalg.norm(ref))
    if nz == 1:
        assert (err <= 1.125 * U * np.abs(ref)).all(), float((err / np.abs(ref)).max() / U)


@pytest.mark.parametrize("n,fin,fout,offset", [(500, 70, 40, 0), (700, 300, 130, 1), (66001, 40, 16, 0),
                                               (66000, 33, 31, 3), (40003, 100, 200, 0), (70001, 65, 64, 1)])
def test_linear_scattered_infinities_in_every_tile(n, fin, fout, offset):
    """Whole rows and single elements that are not finite, in the first, a
    middle and the last rows and columns of every tile width."""
    X, W = _xw(n, fin, fout)
    rng = np.random.default_rng(5)
    X[rng.integers(0, n, 40), rng.integers(0, fin, 40)] = np.inf
    X[rng.integers(0, n, 40), rng.integers(0, fin, 40)] = -np.inf
    X[n - 1, fin - 1], X[0, 0], X[n // 2] = np.nan, -np.inf, np.nan
    X[17:33] = -np.finfo(np.float32).max      # past bf16's largest; sums overflow
    W[fin - 1, fout - 1], W[0, 0] = np.inf, -np.inf
    wb = torch.zeros(fin * (fout + 1) + offset, device=DEV)
    Wd = wb[offset:].view(fin, fout + 1)[:, :fout]
    Wd.copy_(_dev(W))
    H = agcn.linear(_dev(X), Wd).cpu().numpy()
    rows = np.r_[0:17, 33:n]
    _check(X[rows], W, H[rows])
    # sums of values near the largest may pass infinity on the way: where no
    # order of the sum can, they are the products' sums
    with np.errstate(over="ignore", invalid="ignore"):
        fits = np.abs(X[17:33].astype(np.float64)) @ np.abs(W.astype(np.float64)) < 3.4e38
        ref = X[17:33].astype(np.float64) @ W.astype(np.float64)
        S = np.abs(X[17:33].astype(np.float64)) @ np.abs(W.astype(np.float64))
        assert (np.abs(H[17:33] - ref)[fits] <= ((fin + 12) * U * S)[fits]).all()
        assert not np.isfinite(H[17:33][:, [0, fout - 1]]).any()


def test_linear_of_nan_takes_the_time_of_an_fp32_product():
    """A matrix of NaN (a diverged layer) costs a few times the finite product,
    not a serial sum per element (which took 160 times as long)."""
    n, fin, fout = 20000, 602, 256
    W = torch.randn(fin, fout, device=DEV)
    H = torch.empty(n, fout, device=DEV)

    def best(X):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            agcn.linear(X, W, out=H)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    finite = best(torch.randn(n, fin, device=DEV))
    nan = best(torch.full((n, fin), float("nan"), device=DEV))
    assert torch.isnan(H).all()
    assert nan < 12 * finite, (nan, finite)


def _scaled(rng, shape, exponent):
    return np.ldexp(rng.uniform(1.0, 2.0, shape) * rng.choice([-1.0, 1.0], shape), exponent).astype(np.float32)


@pytest.mark.parametrize("n,fin,fout", [(600, 70, 40), (500, 300, 130), (20001, 70, 40), (40000, 33, 64),
                                        (20000, 100, 150), (3000, 40, 7), (70000, 31, 16)])
def test_linear_of_tiny_values(n, fin, fout):
    """Values whose third parts fall below bf16's smallest number, with factors that
    bring the product back to ordinary size: the fp32 bound relative to |X||W|
    holds for rows that are all tiny, rows that mix tiny and ordinary values,
    columns of tiny weights, and products near and below the smallest normal."""
    rng = np.random.default_rng(fin + fout)
    for ex, ew in [(-103, 60), (-104, 60), (-109, 100), (-112, 100), (-120, 100), (-126, 90), (-135, 120),
                   (-60, -60), (-62, -63), (-63, -63), (-66, -66), (-100, 0)]:
        X, W = _scaled(rng, (n, fin), ex), _scaled(rng, (fin, fout), ew)
        if n % 2 == 0:
            X[::3] *= rng.random((X[::3].shape)) < 0.03       # few nonzeros, and rows of zeros
        _check(X, W, agcn.linear(_dev(X), _dev(W)).cpu().numpy())
        _check(W.T.copy(), X[:fout].T.copy(), agcn.linear(_dev(W.T), _dev(X[:fout].T)).cpu().numpy())
    # tiny values that meet large weights beside ordinary ones that meet small weights
    X, W = _scaled(rng, (n, fin), 0), _scaled(rng, (fin, fout), -30)
    X[1::4, ::3], W[::3, 1::5] = _scaled(rng, X[1::4, ::3].shape, -118), _scaled(rng, W[::3, 1::5].shape, 100)
    W[:, 0] = _scaled(rng, fin, -122)
    W[5, 3], X[2, 7] = 1e-40, 1e-41
    _check(X, W, agcn.linear(_dev(X), _dev(W)).cpu().numpy())
