"""The coarse product where the last coarse value is infinite and the others are
not: the result is P times the infinities that the signs of A_c^{-1}'s last
column give, and the tiles' places past the last unknown add nothing to it.
Coarse spaces of one to ten tiles of 64 unknowns (one launch) and past 640 (two
launches), none a multiple of 64."""
import numpy as np
import pytest

from _cases import gpu_setup_tpfa, tpfa_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block", [((32, 32), 8), ((63, 60), 6), ((150, 140), 6),
                                        ((170, 150), 6)], ids=str)
def test_infinite_last_value(dims, block):
    import torch
    cfg = tpfa_inputs("c1", dims=dims, block=block)
    s, _, _ = gpu_setup_tpfa(cfg, kmax=40)
    n, sup = dims[0] * dims[1], cfg["supports"]
    rp, ci, pv = s.get_prolongation()
    # the corner cell is in the last coarse function's support only
    assert list(ci[rp[-2]:]) == [sup["nc"] - 1] and sup["nc"] % 64 != 0 and np.all(pv > 0)
    v = torch.ones(n, dtype=torch.float64, device="cuda")
    v[-1] = np.inf
    z = torch.empty_like(v)
    s.apply(v, z, pre=(0, 0), post=(0, 0))
    col = np.linalg.inv(s.get_coarse_matrix())[:, -1]
    assert np.abs(col).min() > 1e-12 * np.abs(col).max()      # no sign is rounding
    with np.errstate(invalid="ignore"):
        want = np.add.reduceat(pv * (np.inf * col)[ci], rp[:-1])
    assert np.isposinf(want).sum() > n // 2
    assert np.array_equal(z.cpu().numpy(), want, equal_nan=True)
