"""The 2D tile forms inside PCG (update with two sweeps and residual; prolongation
with sweeps and products) on operators that are not symmetric, whose lower
diagonals are read from their own streams: five and nine neighbours, one work-
group of tiles and ragged grids, one and two sweeps after, against the oracle.

The operator is a symmetric M-matrix whose entries differ by up to 2 per mille
from their transposed ones, so that flexible CG still converges; both sides take
the same steps, and their residuals differ by the amplified rounding of at most
40 of them, below 1e-10."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import synth

pytestmark = pytest.mark.gpu


def _operator(nx, ny, nine, rng):
    n = nx * ny
    i = np.arange(n)
    x, y = i % nx, i // nx
    r, c = [], []
    for dx, dy in ((1, 0), (0, 1), (1, 1), (-1, 1)) if nine else ((1, 0), (0, 1)):
        ok = (x + dx >= 0) & (x + dx < nx) & (y + dy < ny)
        r.append(i[ok])
        c.append((i + dx + nx * dy)[ok])
    r, c = np.concatenate(r), np.concatenate(c)
    U = sp.csr_matrix((-rng.uniform(0.3, 1.0, r.size), (r, c)), shape=(n, n))
    A = (U + U.T).tocsr()
    A = (A + sp.diags(1.1 * np.asarray(abs(A).sum(axis=1)).ravel() + 0.05)).tocsr()
    A.sort_indices()
    off = A.indices != np.repeat(i, np.diff(A.indptr))
    A.data[off] *= 1.0 + 1e-3 * rng.uniform(-1.0, 1.0, off.sum())
    return A


@pytest.mark.parametrize("post", [1, 2])
@pytest.mark.parametrize("nine", [False, True], ids=["five", "nine"])
@pytest.mark.parametrize("dims", [(64, 48), (61, 53), (29, 131), (150, 17)], ids=str)
def test_against_oracle(dims, nine, post):
    import torch
    from paper_1912_06934_amd import Msrsb
    rng = np.random.default_rng(dims[0])
    A = _operator(*dims, nine, rng)
    rp, ci, a = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    sup = synth.make_config("c1", dims=dims, block=7)["supports"]
    coarse = (sup["nc"], sup["part"], sup["prp"], sup["pci"], sup["interior"])
    m, s = oracle.Msrsb(rp, ci, a), Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    for h in (m, s):
        h.set_coarse(*coarse)
    m.setup_basis(kmax=5)
    s.setup_basis(max_iter=5)
    m.build_coarse()
    s.build_coarse()
    f = rng.standard_normal(rp.size - 1)
    ref = m.solve(f, rtol=1e-8, maxit=40, pre=(2, 2), post=(2, post), use_ms=True, hist_cap=41)
    u = torch.zeros(f.size, dtype=torch.float64, device="cuda")
    r = s.solve(torch.from_numpy(f).cuda(), u, rtol=1e-8, max_iter=40, pre=(2, 2), post=(2, post),
                history_cap=41)
    assert r["iters"] == ref["iters"] and 3 <= r["iters"] < 40
    np.testing.assert_allclose(r["history"], ref["hist"][:r["iters"] + 1], rtol=0, atol=1e-10)
    assert np.max(np.abs(u.cpu().numpy() - ref["x"])) <= 1e-9 * np.max(np.abs(ref["x"]))
