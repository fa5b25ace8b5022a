"""2D grids on either side of the lines where the tile forms stop paying: the
basis in both precisions against the oracle (512 and 522 tiles of nine
neighbours, five neighbours with tiles up to 1.9 times the grid), and the FP32
smoother inside PCG on a long narrow grid (up to 200,000 rows in tiles).

Tolerances as for the smaller grids: 1e-12 in FP64 and 1e-4 in FP32 after 12
steps of sums of at most nine products, and the solution's own residual."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_tile_smoothing import _operator

pytestmark = pytest.mark.gpu


def _supports(nx, ny, block):
    sup = synth.cell_supports((nx, ny), block)
    return tuple(sup[q] for q in ("nc", "part", "prp", "pci", "interior"))


@pytest.mark.parametrize("nx,ny,nine", [(25, 6144, True), (25, 6250, True), (25, 12288, False),
                                        (25, 13000, False)], ids=str)
def test_basis(nx, ny, nine):
    from paper_1912_06934_amd import Msrsb
    A = _operator(nx, ny, nine, False, False, np.random.default_rng(ny))
    rp, ci, a = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    nc, part, prp, pci, inner = _supports(nx, ny, 25)
    s = Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    s.set_coarse(nc, part, prp, pci, inner)
    jv, _ = oracle.filter_jacobi(rp, ci, a)
    pv, it, e, _ = oracle.basis(rp, ci, jv, prp, pci, oracle.init_basis(prp, pci, part), inner,
                                kmax=12)
    for fp32, tol in ((False, 1e-12), (True, 1e-4)):
        info = s.setup_basis(max_iter=12, fp32_basis=fp32)
        assert info["iters"] == it and abs(info["e_it"] - e) <= tol
        assert np.max(np.abs(s.get_prolongation()[2] - pv)) <= tol


@pytest.mark.parametrize("ny", [12500, 12501])
@pytest.mark.parametrize("nine", [False, True], ids=["five", "nine"])
def test_fp32_smoother(ny, nine):
    import torch
    from paper_1912_06934_amd import Msrsb
    A = _operator(16, ny, nine, False, False, np.random.default_rng(4))
    n = A.shape[0]
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    s.set_coarse(*_supports(16, ny, 16))
    s.setup_basis(max_iter=10)
    s.build_coarse()
    f = np.random.default_rng(1).standard_normal(n)
    iters = {}
    for fp32 in (False, True):
        u = torch.zeros(n, dtype=torch.float64, device="cuda")
        r = s.solve(torch.from_numpy(f).cuda(), u, rtol=1e-10, max_iter=200, pre=(2, 2),
                    post=(2, 1), fp32_smoother=fp32)
        iters[fp32] = r["iters"]
        assert r["true_rel_res"] <= 1e-10
        assert np.linalg.norm(f - A @ u.cpu().numpy()) <= 1.1e-10 * np.linalg.norm(f)
    # (an FP32 preconditioner is the same up to 1e-7: a step more at most)
    assert abs(iters[False] - iters[True]) <= 1
