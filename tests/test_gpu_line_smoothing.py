"""The smoothing of P for operators of 27 diagonals in lines of three against
the oracle: row counts around the work-group's 256 rows, grids whose lines are
shorter and longer than that, one and three components per node, symmetric
(factored J, scalar) and unsymmetric values, absent couplings, checked steps.

Tolerance: a step adds at most 27 products and divides by a row sum of order
one, so 25 steps differ by 1e-12 at most (FP32: the same argument with its
precision, 1e-4)."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import synth
from synth.grids import vector_supports

pytestmark = pytest.mark.gpu


def _operator(dims, bs, unsym, rng):
    nx, ny, nz = dims
    nn = nx * ny * nz
    idx = np.arange(nn)
    x, y, z = idx % nx, idx // nx % ny, idx // (nx * ny)
    r, c = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dz, dy, dx) <= (0, 0, 0):
                    continue
                ok = (x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz < nz)
                ok &= rng.uniform(size=nn) < 0.97  # some couplings are absent
                ok[:2] = (x + dx >= 0)[:2] & (x + dx < nx)[:2] & (y + dy >= 0)[:2] & (
                    y + dy < ny)[:2] & (z + dz < nz)[:2]
                r.append(idx[ok])
                c.append(idx[ok] + dx + nx * dy + nx * ny * dz)
    r, c = np.concatenate(r), np.concatenate(c)
    U = sp.coo_matrix((-rng.uniform(0.1, 1.0, r.size), (r, c)), shape=(nn, nn)).tocsr()
    A = U + U.T
    A = (A + sp.diags(1.1 * np.asarray(abs(A).sum(axis=1)).ravel())).tocsr()
    if bs > 1:
        B = np.eye(bs) + 0.2 * np.ones((bs, bs))
        A = sp.kron(A, B).tocsr()
    if unsym:
        A.data *= rng.uniform(0.9, 1.1, A.data.size)
    A.sort_indices()
    return A


@pytest.mark.parametrize("dims,block,bs", [((7, 6, 5), 3, 1), ((8, 8, 4), 4, 1), ((257, 4, 3), 5, 1),
                                           ((16, 16, 16), 4, 1), ((5, 17, 3), 3, 3),
                                           ((300, 3, 4), 6, 3), ((12, 11, 10), 4, 3),
                                           ((43, 3, 2), 4, 3)], ids=str)
@pytest.mark.parametrize("unsym", [False, True], ids=["symmetric", "unsymmetric"])
def test_line_smoothing(dims, block, bs, unsym):
    from paper_1912_06934_amd import Msrsb
    A = _operator(dims, bs, unsym, np.random.default_rng(sum(dims)))
    rp, ci, a = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    sup = synth.cell_supports(dims, block)
    if bs > 1:
        sup = vector_supports(sup, bs)
    nc, part, prp, pci, inner = (sup[q] for q in ("nc", "part", "prp", "pci", "interior"))
    s = Msrsb(device=0)
    s.set_matrix(rp, ci, a, bs)
    s.set_coarse(nc, part, prp, pci, inner)
    jv, _ = oracle.filter_jacobi(rp, ci, a, bs)
    pv0 = oracle.init_basis(prp, pci, part)
    for kmax, tol, every in ((25, -1.0, 1), (25, 1e-3, 4)):
        pv, it, e, _ = oracle.basis(rp, ci, jv, prp, pci, pv0, inner, kmax=kmax,
                                    tol=tol, nit=every)
        info = s.setup_basis(max_iter=kmax, tol=tol, check_every=every)
        assert info["iters"] == it
        assert np.max(np.abs(s.get_prolongation()[2] - pv)) <= 1e-12
        assert abs(info["e_it"] - e) <= 1e-12
    s.setup_basis(max_iter=25, fp32_basis=True)
    pv = oracle.basis(rp, ci, jv, prp, pci, pv0, inner, kmax=25)[0]
    assert np.max(np.abs(s.get_prolongation()[2] - pv)) <= 1e-4
