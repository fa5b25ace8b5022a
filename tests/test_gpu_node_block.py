"""Sweeps of the node-block (3 components, 27 node offsets) operator against
plain sparse algebra: symmetric values (mirrored upper entries) and row-scaled
non-symmetric ones (all entries), on grids around one wavefront of nodes and on
both sides of the three-threads-per-node limit (131,072 nodes).

Tolerances: a row sums 81 products, so two FP64 evaluations of two l1-Jacobi
sweeps differ by at most a few hundred roundings of 1.1e-16: 1e-13 of the
largest entry; FP32 values and arithmetic, 81 roundings of 6e-8 per sweep:
2e-5."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

L1 = 2


def _sweeps(s, v, fp32):
    import torch
    z = torch.empty(v.size, dtype=torch.float64, device="cuda")
    s.apply(torch.from_numpy(v).cuda(), z, pre=(L1, 2), post=(0, 0), use_multiscale=False,
            fp32_smoother=fp32)
    return z.cpu().numpy()


@pytest.mark.parametrize("elems,symmetric", [
    ((3, 3, 3), True), ((3, 3, 3), False),        # 64 nodes: one wavefront
    ((2, 2, 6), True), ((2, 2, 6), False),        # 63
    ((4, 12, 2), True),                           # 195: three wavefronts and three nodes
    ((19, 8, 11), True), ((19, 8, 11), False),
    ((43, 44, 44), True), ((43, 44, 44), False),  # 89,100: seven threads per node
    ((44, 44, 44), True),                         # 91,125: one
    ((51, 51, 47), True),                         # 129,792
    ((51, 51, 48), True), ((51, 51, 48), False),  # 132,496
], ids=lambda x: str(x))
def test_sweeps_match_sparse_algebra(elems, symmetric):
    from paper_1912_06934_amd import Msrsb
    rng = np.random.default_rng(7)
    s = Msrsb(device=0)
    nodes = [e + 1 for e in elems]
    n = 3 * int(np.prod(nodes))
    fixed = np.zeros(n, dtype=np.uint8)
    fixed[:3 * nodes[0] * nodes[1]] = 1
    s.assemble_q1(elems, (0.3, 0.2, 0.25), 0.3, 0.5 * rng.standard_normal(int(np.prod(elems))),
                  fixed)
    assert s.n == n
    rp, ci, a = s.get_matrix()
    if not symmetric:
        a = a * np.repeat(rng.uniform(0.5, 2.0, n), np.diff(rp))
        s.set_matrix(rp, ci, a, 3)
    A = sp.csr_matrix((a, ci, rp), shape=(n, n))
    d = 1.0 / np.asarray(abs(A).sum(axis=1)).ravel()
    v = rng.standard_normal(n)
    z = d * v
    z = z + d * (v - A @ z)
    for fp32, tol in ((False, 1e-13), (True, 2e-5)):
        got = _sweeps(s, v, fp32)
        assert np.max(np.abs(got - z)) <= tol * np.max(np.abs(z))
