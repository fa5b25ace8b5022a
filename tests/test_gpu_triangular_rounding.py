"""The triangular solves divide by the pivots: a quotient of exactly known
numbers is the correctly rounded one, on each form of the solves (one
wavefront, one work-group, a launch per level, rows that end in the first pass
and in the second), and an infinite pivot gives a zero.

Blocks of two rows [[p, q], [k p, d + k q]] with whole p, q, k have the ILU(0)
factors l = k, u = [[p, q], [0, d]] without rounding.  For b = (b0, k b0 + b1)
the second row's result is b1 / d.  With q = 0 the first row's is b0 / p.  For
IC(0) a diagonal matrix of squares d^2 gives b / d / d, two roundings."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

ILU0, SGS, IC0 = 3, 4, 5


def _apply(A, b, kind, order):
    import torch
    from paper_1912_06934_amd import Msrsb
    A.sort_indices()
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    z = torch.full((b.size,), np.nan, dtype=torch.float64, device="cuda")
    s.apply(torch.from_numpy(b).cuda(), z, pre=(0, 0), post=(kind, 1), use_multiscale=False,
            ordering=order)
    return z.cpu().numpy()


def _blocks(pairs, stride, rng, upper):
    """Blocks on the rows i, i + stride."""
    n = 2 * pairs
    i = np.arange(pairs)
    first = i // stride * 2 * stride + i % stride
    p = rng.integers(3, 2000, pairs).astype(np.float64)
    d = rng.integers(3, 2000, pairs).astype(np.float64)
    k = rng.integers(1, 9, pairs).astype(np.float64)
    q = rng.integers(1, 9, pairs) * float(upper)
    r = np.concatenate([first, first, first + stride, first + stride])
    c = np.concatenate([first, first + stride, first, first + stride])
    A = sp.csr_matrix((np.concatenate([p, q, k * p, d + k * q]), (r, c)), shape=(n, n))
    b0 = rng.integers(1, 10**6, pairs).astype(np.float64)
    b1 = rng.integers(1, 10**6, pairs).astype(np.float64)
    b = np.empty(n)
    b[first], b[first + stride] = b0, k * b0 + b1
    return A, b, first, first + stride, b0 / p, b1 / d


FORMS = [(40, 40, "natural"),        # one wavefront
         (120, 120, "natural"),      # one wavefront, two rows per lane
         (1000, 1000, "natural"),    # one work-group, x in LDS
         (9000, 1000, "natural"),    # ... past LDS
         (3000, 3000, "natural"),    # a launch per level
         (1000, 1, "multicolor"), (3000, 1, "multicolor")]


@pytest.mark.parametrize("pairs,stride,order", FORMS, ids=str)
def test_quotients_are_correctly_rounded(pairs, stride, order):
    rng = np.random.default_rng(pairs)
    A, b, _, second, _, quot = _blocks(pairs, stride, rng, True)
    assert np.array_equal(_apply(A, b, ILU0, order)[second], quot)
    A, b, first, second, quot0, quot1 = _blocks(pairs, stride, rng, False)
    z = _apply(A, b, ILU0, order)
    assert np.array_equal(z[first], quot0) and np.array_equal(z[second], quot1)
    # (a diagonal matrix is solved by the forward half sweep; with exact quotients
    # the backward one adds nothing)
    n = b.size
    d = rng.integers(3, 2000, n).astype(np.float64)
    D = sp.diags(d * d).tocsr()
    assert np.array_equal(_apply(D, b, IC0, order), b / d / d)
    z = _apply(sp.diags(d).tocsr(), d * np.floor(b), SGS, order)
    assert np.array_equal(z, np.floor(b))


@pytest.mark.parametrize("pairs,stride,order", FORMS, ids=str)
def test_infinite_pivots(pairs, stride, order):
    rng = np.random.default_rng(pairs)
    A, b, first, second, quot0, quot1 = _blocks(pairs, stride, rng, False)
    A.sort_indices()
    diag = np.flatnonzero(A.indices == np.repeat(np.arange(b.size), np.diff(A.indptr)))
    A.data[diag[second[::3]]] = np.inf
    z = _apply(A, b, ILU0, order)
    quot1 = quot1.copy()
    quot1[::3] = 0.0
    assert np.array_equal(z[first], quot0) and np.array_equal(z[second], quot1)


@pytest.mark.parametrize("pairs,stride,order", FORMS, ids=str)
def test_infinite_values(pairs, stride, order):
    rng = np.random.default_rng(pairs)
    A, b, first, second, quot0, quot1 = _blocks(pairs, stride, rng, False)
    b[second[::5]] = -np.inf
    z = _apply(A, b, ILU0, order)
    quot1 = quot1.copy()
    quot1[::5] = -np.inf
    assert np.array_equal(z[second], quot1)
    # (the first row of a block holds its stored zero times the second's result)
    assert np.array_equal(np.delete(z[first], np.s_[::5]), np.delete(quot0, np.s_[::5]))


@pytest.mark.parametrize("kind", [ILU0, IC0], ids=["ilu0", "ic0"])
@pytest.mark.parametrize("grid,stencil,order", [
    ((64, 64, 1), "box", "natural"), ((40, 40, 12), "star", "natural"),
    ((70, 64, 60), "star", "natural"), ((97, 89, 1), "star", "multicolor"),
    ((97, 89, 1), "box", "multicolor"), ((28, 27, 25), "box", "multicolor")], ids=str)
def test_infinities_spread_as_in_the_sequential_solve(grid, stencil, order, kind):
    """Rows with fewer entries than their level's widest: what fills them must
    not meet an infinite value.  The oracle's solves add each stored entry in
    turn; with entries of one sign an infinite value spreads and gives no NaN."""
    import oracle
    from test_gpu_triangular import _grid
    rng = np.random.default_rng(7)
    rp, ci, a = _grid(*grid, stencil, rng, True)
    n = rp.size - 1
    b = rng.standard_normal(n)
    few = np.flatnonzero(np.diff(rp) < np.diff(rp).max())
    b[few[2 * few.size // 3]] = np.inf
    m = oracle.Msrsb(rp, ci, a)
    one = np.zeros(n, dtype=np.int32)
    m.set_coarse(1, one, np.arange(n + 1, dtype=np.int32), one, np.ones(n, dtype=np.uint8))
    m.setup_basis(kmax=1)
    m.build_coarse()
    ref = m.apply(b, pre=(0, 0), post=(kind, 1), use_ms=False, ordering=order)
    z = _apply(sp.csr_matrix((a, ci, rp), shape=(n, n)), b, kind, order)
    ok = np.isfinite(ref)
    assert not ok.all() and np.all(ref[~ok] == np.inf)
    np.testing.assert_array_equal(z[~ok], ref[~ok])
    np.testing.assert_allclose(z[ok], ref[ok], rtol=0, atol=1e-12 * np.abs(b[np.isfinite(b)]).max())
