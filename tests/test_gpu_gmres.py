"""GMRES against the oracle's residual history on the forms its
orthogonalisation takes: columns up to 8, 16 and 32 (four launches a step) and
past 32 (a launch per operation), rows around one work-group (512) and past 256
work-groups (131,072: two rows per thread).

Tolerance: the matrix has a condition number below 40, so the rounding of the
Krylov basis (1e-16 per operation, at most a few hundred of them) moves the
relative residuals by less than 1e-11 absolute."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle

pytestmark = pytest.mark.gpu

JACOBI, ILU0 = 1, 3


def _matrix(n, rng):
    d = np.arange(n)
    A = sp.diags([3.0 + np.cos(d), -1.0 - 0.3 * rng.random(n - 1), -0.4 * rng.random(n - 1),
                  -0.3 * rng.random(n - 7)], [0, -1, 1, 7]).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data


@pytest.mark.parametrize("n,restart,kind", [
    (511, 5, JACOBI), (512, 8, JACOBI), (513, 9, ILU0), (700, 16, JACOBI), (3000, 17, JACOBI),
    (1025, 32, JACOBI), (5000, 33, JACOBI), (3000, 64, JACOBI), (131072, 20, JACOBI),
    (131073, 20, JACOBI), (300007, 40, JACOBI), (64, 1, JACOBI),
])
def test_residual_history(n, restart, kind):
    import torch
    from paper_1912_06934_amd import Msrsb
    rng = np.random.default_rng(n)
    rp, ci, a = _matrix(n, rng)
    f = rng.standard_normal(n)
    m = oracle.Msrsb(rp, ci, a)
    one = np.zeros(n, dtype=np.int32)             # a coarse space of one node, not used
    m.set_coarse(1, one, np.arange(n + 1, dtype=np.int32), one, np.ones(n, dtype=np.uint8))
    m.setup_basis(kmax=1)
    m.build_coarse()
    ref = m.solve(f, krylov="gmres", restart=restart, rtol=1e-11, maxit=400, pre=(0, 0),
                  post=(kind, 1), use_ms=False, hist_cap=500)
    s = Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    u = torch.zeros(n, dtype=torch.float64, device="cuda")
    r = s.solve(torch.from_numpy(f).cuda(), u, krylov="gmres", restart=restart, rtol=1e-11,
                max_iter=400, post=(kind, 1), use_multiscale=False, history_cap=500)
    assert abs(r["iters"] - ref["iters"]) <= 1
    k = min(r["iters"], ref["iters"])
    np.testing.assert_allclose(r["history"][:k], ref["hist"][:k], rtol=0, atol=1e-11)
    x = ref["x"]
    assert np.max(np.abs(u.cpu().numpy() - x)) <= 1e-9 * np.max(np.abs(x))
