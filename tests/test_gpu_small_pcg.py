"""PCG on small stencil problems (one work-group) against the oracle: sizes
around a wavefront, the rows per thread (1024 a row), the largest one (2048 rows,
64 coarse unknowns) and past it, with
one, five, seven and nine diagonals, narrow and wide rows of P, sweeps on either
side, without the coarse stage, from a non-zero start, through the transposed
entry; and more steps than one launch takes.

Tolerance: condition numbers below 100 and at most a hundred steps; the two
sides' relative residuals differ by the amplified rounding of the recurrences,
below 1e-10 absolute."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from _cases import tpfa_inputs

pytestmark = pytest.mark.gpu

NONE, JACOBI, L1 = 0, 1, 2


def _stencil(n, offs, rng):
    """SPD with the given upper offsets (those that fit), diagonally dominant."""
    U = sp.csr_matrix((n, n))
    for o in offs:
        if o < n:
            U = U + sp.diags(-rng.uniform(0.3, 1.0, n - o), o, shape=(n, n))
    A = U + U.T
    A = (A + sp.diags(1.1 * np.asarray(abs(A).sum(axis=1)).ravel() + 0.05)).tocsr()
    A.sort_indices()
    return A


def _coarse(n, blocks, wide):
    """Blocks of consecutive rows, each one's support reaching into its
    neighbours (wide: further, up to 8 supports a row)."""
    per = -(-n // blocks)
    part = np.arange(n) // per
    nc = int(part[-1]) + 1
    reach = 3 if wide else 1
    prp, pci = [0], []
    for i in range(n):
        c = [j for j in range(part[i] - reach, part[i] + reach + 1) if 0 <= j < nc]
        pci += c
        prp.append(len(pci))
    return (nc, part.astype(np.int32), np.array(prp, np.int32), np.array(pci, np.int32),
            np.ones(n, np.uint8))


def _check(A, coarse, pre, post, ms, x0=None, trans=False, rtol=1e-11):
    import torch
    from paper_1912_06934_amd import Msrsb, MsrsbError
    n = A.shape[0]
    rp, ci, a = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    f = np.random.default_rng(n).standard_normal(n)
    m, s = oracle.Msrsb(rp, ci, a), Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    for h in (m, s):
        h.set_coarse(*coarse)
    m.setup_basis(kmax=3)
    s.setup_basis(max_iter=3)
    m.build_coarse()
    s.build_coarse()
    g = f if x0 is None else f - A @ x0
    # (from x0 the oracle solves for the correction, to the same threshold)
    scale = np.linalg.norm(f) / np.linalg.norm(g)
    ref = m.solve(g, rtol=rtol * scale, maxit=300, pre=post if trans else pre,
                  post=pre if trans else post, use_ms=ms, hist_cap=400)
    x = ref["x"] if x0 is None else x0 + ref["x"]
    fd = torch.from_numpy(f).cuda()
    u = torch.zeros_like(fd) if x0 is None else torch.from_numpy(x0).cuda()
    go = s.solve_transpose if trans else s.solve
    kw = dict(rtol=rtol, pre=pre, post=post, use_multiscale=ms, history_cap=400)
    r = go(fd, u, max_iter=300, **kw)
    assert abs(r["iters"] - ref["iters"]) <= 1
    assert r["true_rel_res"] <= rtol
    k = min(r["iters"], ref["iters"])
    np.testing.assert_allclose(r["history"][:k], ref["hist"][:k] / scale, rtol=0, atol=1e-10)
    assert np.max(np.abs(u.cpu().numpy() - x)) <= 1e-9 * np.max(np.abs(x))
    if ref["iters"] > 3:
        u.zero_() if x0 is None else u.copy_(torch.from_numpy(x0))
        with pytest.raises(MsrsbError) as e:
            go(fd, u, max_iter=3, **kw)
        assert e.value.name == "MSRSB_E_NOT_CONVERGED" and e.value.info["iters"] == 3
        np.testing.assert_allclose(e.value.info["history"], ref["hist"][:4] / scale, rtol=0,
                                   atol=1e-10)
        assert abs(e.value.info["true_rel_res"] - ref["hist"][3] / scale) <= 1e-10


@pytest.mark.parametrize("n,offs,wide", [
    (1, (), False), (2, (1,), False), (63, (1,), False), (64, (1, 8), True), (65, (1, 8), False),
    (1000, (1, 37), False), (1023, (1, 30), True), (1024, (1, 7, 80), True),
    (1025, (1, 7, 80, 81), False), (1984, (1, 44), False), (2015, (1, 44), True), (2048, (1, 45), False), (2049, (1, 13, 200), True),
    (4095, (1, 60, 61, 62), True), (4096, (1, 64), False), (4096, (1, 16, 256), True),
    (4097, (1, 64), False)], ids=str)
@pytest.mark.parametrize("pre,post,ms", [((NONE, 0), (JACOBI, 1), True), ((L1, 2), (L1, 2), True),
                                         ((JACOBI, 1), (L1, 3), False)], ids=str)
def test_against_oracle(n, offs, wide, pre, post, ms):
    A = _stencil(n, offs, np.random.default_rng(n + 1))
    _check(A, _coarse(n, max(1, min(n // (31 if n in (1984, 2015) else 40), 250)), wide), pre, post, ms)


@pytest.mark.parametrize("pre,post,trans", [((L1, 1), (L1, 1), False), ((L1, 1), (NONE, 0), True),
                                            ((NONE, 0), (L1, 2), True)], ids=str)
def test_start_and_transpose(pre, post, trans):
    rng = np.random.default_rng(0)
    n = 1500
    A = _stencil(n, (1, 40), rng)
    _check(A, _coarse(n, 24, False), pre, post, True, x0=rng.standard_normal(n), trans=trans)


@pytest.mark.parametrize("dims", [(32, 32), (17, 13, 11)], ids=str)
def test_flow_grids(dims):
    cfg = tpfa_inputs("c1" if len(dims) == 2 else "c5", dims=dims, block=4)
    n = cfg["rp"].size - 1
    A = sp.csr_matrix((cfg["a"], cfg["ci"], cfg["rp"]), shape=(n, n))
    # (scaled to a moderate condition number)
    A = (A + sp.diags(0.2 * A.diagonal())).tocsr()
    A.sort_indices()
    sup = cfg["supports"]
    _check(A, (sup["nc"], sup["part"], sup["prp"], sup["pci"], sup["interior"]), (L1, 2), (L1, 2),
           True)


def test_more_steps_than_a_launch():
    # a 1D Laplacian without a coarse stage needs a step per row; the history
    # runs on from launch to launch: the recurrence's residuals of the steps on
    # both sides of a launch's end (1024) are those of one run
    import torch
    from paper_1912_06934_amd import Msrsb
    n = 2000
    A = sp.diags([-np.ones(n - 1), 2.0 * np.ones(n), -np.ones(n - 1)], [-1, 0, 1]).tocsr()
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    f = np.random.default_rng(1).standard_normal(n)
    u = torch.zeros(n, dtype=torch.float64, device="cuda")
    r = s.solve(torch.from_numpy(f).cuda(), u, rtol=1e-8, max_iter=8000, pre=(NONE, 0),
                post=(JACOBI, 1), use_multiscale=False, history_cap=8001)
    x = u.cpu().numpy()
    assert r["iters"] > 1024 and r["true_rel_res"] <= 1e-8
    assert np.linalg.norm(f - A @ x) <= 1.01e-8 * np.linalg.norm(f)
    h = np.asarray(r["history"])
    assert h.size == r["iters"] + 1 and np.all(np.isfinite(h)) and h[0] == 1.0
    # textbook CG (Jacobi is a scaling here) in the same precision: the early
    # steps agree closely, and no step near the launch's end jumps
    y, res, p = np.zeros(n), f.copy(), f.copy()
    rr, ref = res @ res, [1.0]
    for _ in range(200):
        q = A @ p
        al = rr / (p @ q)
        res = res - al * q
        new = res @ res
        p = res + new / rr * p
        rr = new
        ref.append(np.sqrt(rr) / np.linalg.norm(f))
    np.testing.assert_allclose(h[:201], ref, rtol=1e-6)
    step = np.abs(np.diff(np.log(h[900:1150])))
    assert step[[123, 124, 125]].max() <= 2.0 * step.max() and step[120:130].max() < 1.0


@pytest.mark.parametrize("n,offs,wide", [
    (1, (), False), (64, (1, 8), True), (65, (1, 8), False), (1000, (1, 37), False),
    (1024, (1, 30), True), (1024, (1, 7, 80, 81), True), (1025, (1, 7, 80), True),
    (1025, (1, 7, 80, 81), False), (1900, (1, 45), False), (1937, (1, 13, 200), False),
    (1938, (1, 13, 200), False), (2048, (1, 45), False)], ids=str)
@pytest.mark.parametrize("unsym", [False, True], ids=["symmetric", "unsymmetric"])
def test_smoothing_against_oracle(n, offs, wide, unsym):
    """The basis after a fixed number of steps, checked or not, and to a
    tolerance: the steps add at most nine products, each step divides by a row
    sum of order one, so 40 steps differ by 1e-12 at most (FP32: the same
    argument with its precision, 1e-4)."""
    from paper_1912_06934_amd import Msrsb
    A = _stencil(n, offs, np.random.default_rng(n + 2))
    if unsym:
        A.data *= 1.0 + 0.3 * (A.indices > np.repeat(np.arange(n), np.diff(A.indptr)))
    rp, ci, a = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    coarse = _coarse(n, max(1, min(n // 40, 60)), wide)
    # rows that no check looks at
    coarse[4][::7] = 0
    s = Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    s.set_coarse(*coarse)
    jv, _ = oracle.filter_jacobi(rp, ci, a)
    pv0 = oracle.init_basis(coarse[2], coarse[3], coarse[1])
    for kmax, tol, every in ((1, -1.0, 1), (40, -1.0, 1), (40, -1.0, 7), (40, 1e-2, 1),
                             (40, 1e-2, 3), (5, -1.0, 9)):
        pv, it, e, _ = oracle.basis(rp, ci, jv, coarse[2], coarse[3], pv0, coarse[4], kmax=kmax,
                                    tol=tol, nit=every)
        info = s.setup_basis(max_iter=kmax, tol=tol, check_every=every)
        assert info["iters"] == it
        assert np.max(np.abs(s.get_prolongation()[2] - pv)) <= 1e-12
        if every <= kmax:
            assert abs(info["e_it"] - e) <= 1e-12
    s.setup_basis(max_iter=40, fp32_basis=True)
    pv = oracle.basis(rp, ci, jv, coarse[2], coarse[3], pv0, coarse[4], kmax=40)[0]
    assert np.max(np.abs(s.get_prolongation()[2] - pv)) <= 1e-4
