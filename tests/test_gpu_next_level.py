"""The sparse coarse matrix that a further level works on: formed from whole
coarse neighbourhoods (grids that divide evenly and that do not, coarse grids
down to two nodes an axis) and from the general column lists, equal to the
triple product of the fetched P, symmetric to the bit for a symmetric operator
and left as it is for an unsymmetric one.  What asks for a symmetric matrix is
still refused on that level.  Also the preconditioner applied to device vectors
in place.

Tolerance: each entry sums at most a few thousand products of size below
max|A|; 1e-12 of the largest entry."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from _cases import rel_max, tpfa_inputs

pytestmark = pytest.mark.gpu


def _hole(sup):
    """One cell taken out of one support: that support is no box any more."""
    rows = np.repeat(np.arange(sup["part"].size), np.diff(sup["prp"]))
    e = np.flatnonzero(sup["pci"] != sup["part"][rows])[7]
    sup["pci"] = np.delete(sup["pci"], e)
    sup["prp"] = (sup["prp"] - (np.arange(sup["prp"].size) > rows[e])).astype(np.int32)


def _level(cfg, cdims, unsym, fp32):
    from paper_1912_06934_amd import Msrsb
    a = cfg["a"].copy()
    rows = np.repeat(np.arange(cfg["rp"].size - 1), np.diff(cfg["rp"]))
    if unsym:
        a *= 1.0 + 0.2 * (cfg["ci"] > rows)
        a[cfg["ci"] == rows] *= 1.5
    s = Msrsb(device=0)
    s.set_matrix(cfg["rp"], cfg["ci"], a)
    sup = cfg["supports"]
    s.set_coarse(sup["nc"], sup["part"], sup["prp"], sup["pci"], sup["interior"])
    if cdims:
        s2 = synth.cell_supports(cdims, 2)
        s.set_coarse_level(1, s2["nc"], s2["part"], s2["prp"], s2["pci"], s2["interior"])
    s.setup_basis(max_iter=30, fp32_basis=fp32)
    s.build_coarse()
    n = cfg["rp"].size - 1
    A = sp.csr_matrix((a, cfg["ci"], cfg["rp"]), shape=(n, n))
    return s, A


@pytest.mark.parametrize("unsym", [False, True], ids=["symmetric", "unsymmetric"])
@pytest.mark.parametrize("dims,block,fp32", [((24, 24, 16), 4, False), ((21, 13, 9), 4, False),
                                             ((21, 13, 9), 4, True), ((9, 30, 8), 5, False),
                                             ((8, 9, 10), 5, False)], ids=str)
@pytest.mark.parametrize("boxes", [True, False], ids=["boxes", "holes"])
def test_next_level_matrix(dims, block, fp32, boxes, unsym):
    from paper_1912_06934_amd import MsrsbError
    cfg = tpfa_inputs("c5", dims=dims, block=block)
    if not boxes:
        _hole(cfg["supports"])
    cdims = tuple(-(-d // block) for d in dims)
    s, A = _level(cfg, cdims, unsym, fp32)
    prp, pci, pv = s.get_prolongation()
    nc = cfg["supports"]["nc"]
    P = sp.csr_matrix((pv, pci, prp), shape=(A.shape[0], nc))
    rp, ci, va = s.level(1).get_matrix()
    Ac = sp.csr_matrix((va, ci, rp), shape=(nc, nc)).toarray()
    assert rel_max(Ac, (P.T @ A @ P).toarray()) <= 1e-12
    assert np.array_equal(Ac, Ac.T) == (not unsym)
    # new values through the same pattern
    s.update_values(2.0 * A.data)
    s.setup_basis(max_iter=30, fp32_basis=fp32)
    s.build_coarse()
    Ac2 = sp.csr_matrix((s.level(1).get_matrix()[2], ci, rp), shape=(nc, nc)).toarray()
    assert np.array_equal(Ac2, 2.0 * Ac)
    with pytest.raises(MsrsbError):
        s.build_coarse(factor="cholesky")


@pytest.mark.parametrize("pre,post", [((0, 0), (0, 0)), ((2, 2), (2, 2)), ((1, 1), (0, 0)),
                                      ((3, 1), (1, 2))], ids=str)
def test_apply_device_vectors(pre, post):
    # the result over its input, and from host vectors: the same bits
    import torch
    cfg = tpfa_inputs("c5", dims=(21, 13, 9), block=4)
    # (the triangular kinds are for a finest level without further ones)
    s, A = _level(cfg, None if pre[0] > 2 else (6, 4, 3), False, False)
    v = np.random.default_rng(2).standard_normal(A.shape[0])
    z = np.zeros_like(v)
    s.apply(v, z, pre=pre, post=post)
    d = torch.from_numpy(v).cuda()
    out = torch.full_like(d, float("nan"))
    s.apply(d, out, pre=pre, post=post)
    assert np.array_equal(out.cpu().numpy(), z)
    assert np.array_equal(d.cpu().numpy(), v)
    s.apply(d, d, pre=pre, post=post)
    assert np.array_equal(d.cpu().numpy(), z)


@pytest.mark.parametrize("tol,every,kmax", [(-1.0, 1, 7), (-1.0, 3, 7), (-1.0, 5, 5), (-1.0, 9, 7),
                                            (1e-3, 1, 60), (1e-3, 4, 60)])
def test_last_basis_change(tol, every, kmax):
    # the reported change of the basis: that of the last checked step
    from oracle import basis, filter_jacobi, init_basis
    from paper_1912_06934_amd import Msrsb
    cfg = tpfa_inputs("c5", dims=(12, 10, 8), block=4)
    sup = cfg["supports"]
    s = Msrsb(device=0)
    s.set_matrix(cfg["rp"], cfg["ci"], cfg["a"])
    s.set_coarse(sup["nc"], sup["part"], sup["prp"], sup["pci"], sup["interior"])
    info = s.setup_basis(max_iter=kmax, tol=tol, check_every=every)
    jv, _ = filter_jacobi(cfg["rp"], cfg["ci"], cfg["a"])
    pv0 = init_basis(sup["prp"], sup["pci"], sup["part"])
    ref = basis(cfg["rp"], cfg["ci"], jv, sup["prp"], sup["pci"], pv0, sup["interior"],
                kmax=kmax, tol=tol, nit=every)
    assert rel_max(s.get_prolongation()[2], ref[0]) <= 1e-12
    assert info["iters"] == ref[1]
    if every <= kmax:  # (else no step is checked)
        assert abs(info["e_it"] - ref[2]) <= 1e-12
