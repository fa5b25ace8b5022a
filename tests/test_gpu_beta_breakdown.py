"""PCG whose direction breaks down although its step is finite: with
f = (1, 1, 1, 1, ...) and blocks [[1, -1], [-1, -1]] the Jacobi-preconditioned
residual z = (1, -1, ...) has r.z = 0 and z.A z = n, so the step's alpha is 0
and beta = r.(z - z_old) / (r.z)_old is 0 / 0.  The solve reports the breakdown
of step 1 with the iterate of that step, whether further steps were allowed or
not, on every form that PCG takes: one work-group (up to 2,048 rows), scalars
formed by their consumers (up to 131,072) and one-block sums.  All values are
small whole numbers, so nothing is rounded."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_iter", [1, 2, 50])
@pytest.mark.parametrize("n", [2, 64, 2048, 4096, 131072, 140000])
def test_beta_breaks_down(n, max_iter):
    import torch
    from paper_1912_06934_amd import Msrsb, MsrsbError
    e = -np.ones(n - 1)
    e[1::2] = 0.0
    d = np.tile([1.0, -1.0], n // 2)
    A = sp.diags([e, d, e], [-1, 0, 1], format="csr")
    A.sort_indices()
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    u0 = np.random.default_rng(n).integers(-4, 5, n).astype(np.float64)
    f = torch.from_numpy(A @ u0 + 1.0).cuda()
    u = torch.from_numpy(u0).cuda()
    with pytest.raises(MsrsbError) as err:
        s.solve(f, u, rtol=1e-10, max_iter=max_iter, pre=(0, 0), post=(1, 1),
                use_multiscale=False, history_cap=60)
    assert err.value.name == "MSRSB_E_BREAKDOWN"
    info = err.value.info
    rel = np.sqrt(n) / np.linalg.norm(A @ u0 + 1.0)
    assert info["iters"] == 1
    np.testing.assert_allclose(info["history"], [rel, rel], rtol=1e-14)
    np.testing.assert_allclose(info["true_rel_res"], rel, rtol=1e-14)
    assert np.array_equal(u.cpu().numpy(), u0)
