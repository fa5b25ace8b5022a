"""The triangular smoothers on the forms their solves and factorisations take:
one wavefront (narrow levels in the natural order, one and two rows per lane),
one work-group (levels past 128 rows or rows past four entries a side), a
launch per level (2,048 rows and more, the first two together), patterns that
are not symmetric (no row ends in the first pass), and their limits in rows and
entries, against the oracle's application of the smoother alone.

Tolerance 1e-12 of the largest entry: the factors and solves are the oracle's
operations with reciprocals of the diagonals, the longest dependency chains a
few hundred rows of diagonally dominant matrices, which do not amplify the
rounding of 1.1e-16 per operation."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle

pytestmark = pytest.mark.gpu

ILU0, SGS, IC0 = 3, 4, 5


def _grid(nx, ny, nz, stencil, rng, symmetric):
    """Diagonally dominant matrix on an nx x ny x nz grid: "star" couples along
    the axes, "box" with every neighbour, "up" lacks the entries towards
    larger x (pattern not symmetric)."""
    n = nx * ny * nz
    i = np.arange(n)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    r, c = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dx, dy, dz) == (0, 0, 0):
                    continue
                if stencil != "box" and abs(dx) + abs(dy) + abs(dz) > 1:
                    continue
                if stencil == "up" and dx > 0:
                    continue
                ok = ((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) &
                      (z + dz >= 0) & (z + dz < nz))
                r.append(i[ok])
                c.append((i + dx + nx * (dy + ny * dz))[ok])
    r, c = np.concatenate(r), np.concatenate(c)
    A = sp.csr_matrix((-rng.uniform(0.2, 1.0, r.size), (r, c)), shape=(n, n))
    if symmetric:
        A = 0.5 * (A + A.T)
    A = (A + sp.diags(1.2 * np.asarray(abs(A).sum(axis=1)).ravel() + 0.1)).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data


CASES = [
    # (grid, stencil, symmetric, order): the form
    ((9, 7, 1), "box", True, "natural"),         # one wavefront, a few levels
    ((64, 64, 1), "box", True, "natural"),       # 32 rows a level
    ((40, 300, 1), "star", True, "natural"),     # two entries a side, 40 rows
    ((130, 126, 1), "box", False, "natural"),    # 16,380 rows: x just fits LDS, 63-65 rows a level
    ((128, 128, 1), "star", True, "natural"),    # 16,384 rows, 128 rows a level: two rows per lane
    ((130, 127, 1), "box", False, "natural"),    # 16,510 rows: past LDS, one work-group
    ((12, 11, 10), "box", True, "natural"),      # 13 entries a side: one work-group, x in LDS
    ((40, 40, 40), "star", True, "natural"),     # levels up to 1,200 rows
    ((70, 64, 60), "star", False, "natural"),    # levels past 2,048 rows: launches and runs mixed
    ((70, 80, 1), "box", False, "multicolor"),   # four colours of 1,400 rows: one work-group
    ((97, 89, 1), "box", False, "multicolor"),   # four colours of 2,158 rows: launches
    ((31, 23, 17), "star", True, "multicolor"),  # two colours
    ((28, 27, 25), "box", False, "multicolor"),  # eight colours of 2,363 rows, up to 26 entries
    ((90, 95, 1), "up", False, "natural"),       # pattern not symmetric
    ((120, 95, 1), "up", False, "multicolor"),
]


@pytest.mark.parametrize("kind", [ILU0, SGS, IC0], ids=["ilu0", "sgs", "ic0"])
@pytest.mark.parametrize("grid,stencil,symmetric,order", CASES,
                         ids=["x".join(map(str, c[0])) + "-" + c[1] + "-" + c[3] for c in CASES])
def test_smoother_alone(grid, stencil, symmetric, order, kind):
    import torch
    from paper_1912_06934_amd import Msrsb
    if kind == IC0 and not symmetric:
        pytest.skip("IC(0) takes symmetric matrices")
    rng = np.random.default_rng(5)
    rp, ci, a = _grid(*grid, stencil, rng, symmetric)
    n = rp.size - 1
    s = Msrsb(device=0)
    s.set_matrix(rp, ci, a)
    for scale in (1.0, 0.5):                      # the factors follow the values
        v = rng.standard_normal(n)
        m = oracle.Msrsb(rp, ci, scale * a)
        one = np.zeros(n, dtype=np.int32)         # a coarse space of one node, not used
        m.set_coarse(1, one, np.arange(n + 1, dtype=np.int32), one, np.ones(n, dtype=np.uint8))
        m.setup_basis(kmax=1)
        m.build_coarse()
        for sweeps in (1, 2):                     # from zero, and added to an iterate
            ref = m.apply(v, pre=(kind, sweeps), post=(0, 0), use_ms=False, ordering=order)
            z = torch.empty(n, dtype=torch.float64, device="cuda")
            s.apply(torch.from_numpy(v).cuda(), z, pre=(kind, sweeps), post=(0, 0),
                    use_multiscale=False, ordering=order)
            assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
        s.update_values(0.5 * a)
