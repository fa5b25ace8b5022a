"""GMRES that starts a new cycle because the true residual is above the
tolerance although the estimate met it: the first step of the new cycle reports
its own residual, not the one that a step queued ahead in the cycle before left
behind.

FP32 sweeps make estimate and true residual differ (the preconditioner is linear
up to 6e-8 only), so that such cycles end at different columns for different
tolerances.  A solve from the iterate at the cycle's end takes the same first
step with the same operations, so its residual is the same to the bit."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [30, 64])
def test_first_residual_of_a_new_cycle(restart):
    import torch
    from paper_1912_06934_amd import Msrsb, MsrsbError
    rng = np.random.default_rng(2)
    nx, n = 1800, 3240000  # (a step takes the device far longer than the host to queue two)
    A = sp.diags([rng.uniform(-1, -0.2, n - nx), rng.uniform(-1, -0.2, n - 1),
                  rng.uniform(-1, -0.2, n - 1), rng.uniform(-1, -0.2, n - nx)], [-nx, -1, 1, nx])
    A = (A + sp.diags(1.3 * np.asarray(abs(A).sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    f = torch.from_numpy(rng.standard_normal(n)).cuda()

    def solve(u, max_iter, rtol):
        kw = dict(krylov="gmres", restart=restart, rtol=rtol, max_iter=max_iter, pre=(0, 0),
                  post=(1, 2), fp32_smoother=True, use_multiscale=False, history_cap=300)
        try:
            r = s.solve(f, u, **kw)
        except MsrsbError as e:
            assert e.name == "MSRSB_E_NOT_CONVERGED"
            r = e.info
        return r["history"]

    early = 0  # new cycles after an estimate that met the tolerance
    for rtol in (3e-9, 2e-9, 1e-9, 6e-10):
        u = torch.zeros_like(f)
        full = solve(u, 250, rtol)
        for k in range(1, full.size - 2):
            u.zero_()
            part = solve(u, k, rtol)         # ends with the true residual of step k
            if full[k] != part[k]:
                continue                     # the solve went on in its cycle
            early += k % restart != 0
            one = solve(u, 2, rtol)          # (the last step's entry is the true residual)
            assert one[0] == full[k]
            assert one[1] == full[k + 1], (rtol, k, full[k:k + 3], one)
    assert early >= 3
