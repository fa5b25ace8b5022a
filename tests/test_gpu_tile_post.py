"""PCG on 2D grids, where the prolongation, the post-sweeps and the dot products
run in tiles, against the oracle: whole and partial tiles, five and nine
neighbours, one and two post-sweeps (three take their own launches), no, one and
two pre-sweeps, from a start, through the transposed entry, and an operator that
couples across the lines' ends, which the tiles do not serve; FP32 smoother and
basis by the solution's residual.

Tolerance: condition numbers below 100 and at most a hundred steps; the two
sides' relative residuals differ by the amplified rounding of the recurrences,
below 1e-10 absolute."""
import numpy as np
import pytest

import synth
from test_gpu_small_pcg import _check
from test_gpu_tile_smoothing import _operator

pytestmark = pytest.mark.gpu

NONE, JACOBI, L1 = 0, 1, 2


def _supports(nx, ny, block):
    sup = synth.cell_supports((nx, ny), block)
    return tuple(sup[q] for q in ("nc", "part", "prp", "pci", "interior"))


@pytest.mark.parametrize("nx,ny,wrap", [(56, 48, False), (57, 49, False), (130, 17, False),
                                        (16, 150, False), (250, 187, False), (56, 48, True)],
                         ids=str)
@pytest.mark.parametrize("nine", [False, True], ids=["five", "nine"])
@pytest.mark.parametrize("pre,post,trans,start", [
    ((NONE, 0), (JACOBI, 1), False, False), ((L1, 2), (L1, 2), False, False),
    ((L1, 1), (JACOBI, 2), False, True), ((L1, 1), (L1, 1), True, False),
    ((JACOBI, 3), (L1, 3), False, False)], ids=str)
def test_against_oracle(nx, ny, wrap, nine, pre, post, trans, start):
    rng = np.random.default_rng(nx)
    A = _operator(nx, ny, nine, wrap, False, rng)
    x0 = rng.standard_normal(nx * ny) if start else None
    _check(A, _supports(nx, ny, 8 if nx < 200 else 12), pre, post, True, x0=x0, trans=trans)


@pytest.mark.parametrize("fp32_basis,fp32_smoother", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("pre,post", [((L1, 2), (L1, 2)), ((L1, 1), (L1, 1)), ((NONE, 0), (L1, 2))],
                         ids=str)
def test_fp32_parts(fp32_basis, fp32_smoother, pre, post):
    import torch
    from paper_1912_06934_amd import Msrsb
    A = _operator(90, 61, True, False, False, np.random.default_rng(4))
    n = A.shape[0]
    s = Msrsb(device=0)
    s.set_matrix(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    s.set_coarse(*_supports(90, 61, 8))
    s.setup_basis(max_iter=10, fp32_basis=fp32_basis)
    s.build_coarse()
    f = np.random.default_rng(1).standard_normal(n)
    out = {}
    for fp32 in (False, fp32_smoother):
        u = torch.zeros(n, dtype=torch.float64, device="cuda")
        r = s.solve(torch.from_numpy(f).cuda(), u, rtol=1e-11, max_iter=200, pre=pre, post=post,
                    fp32_smoother=fp32)
        out[fp32] = r["iters"]
        assert r["true_rel_res"] <= 1e-11
        assert np.linalg.norm(f - A @ u.cpu().numpy()) <= 1.1e-11 * np.linalg.norm(f)
    # (an FP32 preconditioner is the same up to 1e-7: a step more at most)
    assert abs(out[False] - out[fp32_smoother]) <= 1
