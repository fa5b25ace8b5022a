"""What is formed from a matrix's values when they are set, for the stencil
storage forms (diagonals; node blocks of 2 and 3 components): the smoothers'
diagonal inverses against the CSR rows (to the last bit: one entry per row
times one), and the symmetry test, seen through IC(0), which takes symmetric
matrices only.  Row counts lie around the work-groups' tiles."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

JACOBI, L1, IC0 = 1, 2, 5


def _stencil(kind, m, rng):
    """A symmetric positive definite matrix of about m rows: CSR and its
    block size."""
    if kind == "tri":                                   # 3 diagonals
        bs, nodes, offs = 1, m, [1]
    elif kind == "dia19":                               # 19 diagonals: the narrow tiles
        bs, nodes, offs = 1, m, list(range(1, 10))
    elif kind == "nb2":                                 # 2 components, node offsets 0, +-1, +-5
        bs, nodes, offs = 2, m // 2, [1, 5]
    else:                                               # 3 components, 27 node offsets
        bs, nodes, offs = 3, m // 3, list(range(1, 14))
    n = bs * nodes
    r, c = [], []
    for o in offs:
        i = np.arange(nodes - o)
        for a in range(bs):
            for b in range(bs):
                r.append(bs * i + a)
                c.append(bs * (i + o) + b)
    i = np.arange(nodes)
    for a in range(bs):
        for b in range(a + 1, bs):
            r.append(bs * i + a)
            c.append(bs * i + b)
    r, c = np.concatenate(r), np.concatenate(c)
    U = sp.csr_matrix((-rng.uniform(0.1, 1.0, r.size), (r, c)), shape=(n, n))
    A = U + U.T
    A = (A + sp.diags(1.0 + np.asarray(abs(A).sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return A, bs


def _solver(A, bs, vals=None):
    from paper_1912_06934_amd import Msrsb
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32),
                 A.data if vals is None else vals, bs)
    return s


def _apply(s, v, pre, fp32=False):
    import torch
    z = torch.empty(v.size, dtype=torch.float64, device="cuda")
    s.apply(torch.from_numpy(v).cuda(), z, pre=pre, post=(0, 0), use_multiscale=False,
            fp32_smoother=fp32)
    return z.cpu().numpy()


CASES = [("tri", 255), ("tri", 257), ("dia19", 127), ("dia19", 130), ("nb2", 62), ("nb2", 130),
         ("nb3", 93), ("nb3", 96), ("nb3", 300)]


@pytest.mark.parametrize("kind,m", CASES)
def test_diagonal_inverses(kind, m):
    A, bs = _stencil(kind, m, np.random.default_rng(m))
    s = _solver(A, bs)
    v = np.ones(A.shape[0])
    l1 = np.zeros(A.shape[0])
    for i in range(A.shape[0]):
        for e in range(A.indptr[i], A.indptr[i + 1]):
            l1[i] += abs(A.data[e])
    d = A.diagonal()
    for code, ref in ((JACOBI, d), (L1, l1)):
        # one multiplication by 1 of a correctly rounded reciprocal
        np.testing.assert_array_equal(_apply(s, v, (code, 1)), 1.0 / ref)
        np.testing.assert_array_equal(_apply(s, v, (code, 1), True),
                                      (1.0 / ref).astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("kind,m", CASES)
def test_symmetry_is_seen_to_the_last_bit(kind, m):
    from paper_1912_06934_amd import MsrsbError
    rng = np.random.default_rng(m)
    A, bs = _stencil(kind, m, rng)
    v = rng.standard_normal(A.shape[0])
    s = _solver(A, bs)
    z = _apply(s, v, (IC0, 1))
    off = np.flatnonzero(np.repeat(np.arange(A.shape[0]), np.diff(A.indptr)) != A.indices)
    for e in (off[0], off[-1], off[off.size // 2]):
        vals = A.data.copy()
        vals[e] = np.nextafter(vals[e], 0.0)
        s.update_values(vals)
        with pytest.raises(MsrsbError):
            _apply(s, v, (IC0, 1))
    s.update_values(A.data)                             # and symmetric again
    np.testing.assert_array_equal(_apply(s, v, (IC0, 1)), z)


@pytest.mark.parametrize("kind,m", [("tri", 200), ("nb3", 96)])
def test_a_stored_zero_without_its_transposed_entry_is_not_symmetric(kind, m):
    from paper_1912_06934_amd import MsrsbError
    rng = np.random.default_rng(m)
    A, bs = _stencil(kind, m, rng)
    C = A.tocoo()
    a, b = 2 * bs, 3 * bs + bs - 1                       # neighbouring nodes
    pair = ((C.row == a) & (C.col == b)) | ((C.row == b) & (C.col == a))
    keep = ~((C.row == b) & (C.col == a))
    data = np.where(pair, 0.0, C.data)
    o = np.lexsort((C.col[keep], C.row[keep]))
    rp = np.zeros(A.shape[0] + 1, dtype=np.int32)
    np.add.at(rp[1:], C.row[keep], 1)
    B = sp.csr_matrix(A.shape)
    B.indptr, B.indices, B.data = np.cumsum(rp).astype(np.int32), C.col[keep][o].astype(np.int32), \
        data[keep][o]
    with pytest.raises(MsrsbError):
        _apply(_solver(B, bs), rng.standard_normal(A.shape[0]), (IC0, 1))


# the coarse product's forms: one launch up to 640 coarse unknowns (11 rows of
# 64 x 64 tiles, ragged last tiles), tiles and sums past that
@pytest.mark.parametrize("blocks", [1, 16, 63, 64, 65, 320, 639, 640, 641, 700])
def test_coarse_product_sizes(blocks):
    """1D, non-overlapping supports: P is the block indicator and the
    preconditioner without smoothing is P A_c^{-1} P^T; A_c is tridiagonal.
    Tolerance: the inverse of a matrix of condition number below 10 and a sum
    of at most 700 products, a few hundred roundings of 1.1e-16."""
    from paper_1912_06934_amd import Msrsb
    import torch
    n = 3 * blocks
    rng = np.random.default_rng(blocks)
    off = -rng.uniform(0.2, 1.0, n - 1)
    A = sp.diags([off, rng.uniform(2.5, 3.0, n), off], [-1, 0, 1]).tocsr()
    A.sort_indices()
    s = _solver(A, 1)
    part = (np.arange(n) // 3).astype(np.int32)
    s.set_coarse(blocks, part, np.arange(n + 1, dtype=np.int32), part, np.ones(n, dtype=np.uint8))
    s.setup_basis(max_iter=1)
    s.build_coarse()
    P = sp.csr_matrix((np.ones(n), part, np.arange(n + 1)), shape=(n, blocks))
    v = rng.standard_normal(n)
    ref = P @ np.linalg.solve((P.T @ A @ P).toarray(), P.T @ v)
    z = torch.empty(n, dtype=torch.float64, device="cuda")
    s.apply(torch.from_numpy(v).cuda(), z, pre=(0, 0), post=(0, 0))
    assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-13 * np.max(np.abs(ref))
