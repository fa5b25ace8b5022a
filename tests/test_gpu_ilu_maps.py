"""ILU(0) in the natural order where most rows lie in wide levels: what the
factorisation keeps for its runs of narrow levels is in proportion to those
runs' rows, and the factors agree with the oracle's through the application of
the smoother alone (1e-12 of the largest entry: a diagonally dominant matrix,
268 levels)."""
import numpy as np
import pytest

import oracle
from test_gpu_triangular import ILU0, _grid

pytestmark = pytest.mark.gpu


def test_memory_of_a_large_grid():
    import torch
    from paper_1912_06934_amd import Msrsb
    rng = np.random.default_rng(5)
    rp, ci, a = _grid(90, 90, 90, "star", rng, False)
    n = rp.size - 1
    v = rng.standard_normal(n)
    vd = torch.from_numpy(v).cuda()
    z = torch.empty_like(vd)
    used = None
    for _ in range(2):                 # (the first time the kernels are loaded as well)
        s = Msrsb(device=0)
        s.set_matrix(rp, ci, a)
        s.apply(vd, z, pre=(1, 1), post=(0, 0), use_multiscale=False)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        s.apply(vd, z, pre=(ILU0, 1), post=(0, 0), use_multiscale=False)
        used = free - torch.cuda.mem_get_info()[0]
    # per entry: side, lower list, transposed place, column, source (17 bytes),
    # the factor and two sets of packed values (24); per row: counts, two rows
    # lists, fold, three sets of diagonals (60); the runs' 43,680 rows at either
    # end of the levels (fewer than 2,048 rows each: the first and last 63) at
    # 256 bytes; 2 MiB of the allocator's grain for each of seven arrays
    bound = 41 * a.size + 60 * n + 256 * 2 * 43680 + 7 * (2 << 20)
    print(f"{used / 2**20:.0f} MiB of at most {bound / 2**20:.0f}", flush=True)
    assert used <= bound
    m = oracle.Msrsb(rp, ci, a)
    one = np.zeros(n, dtype=np.int32)
    m.set_coarse(1, one, np.arange(n + 1, dtype=np.int32), one, np.ones(n, dtype=np.uint8))
    m.setup_basis(kmax=1)
    m.build_coarse()
    ref = m.apply(v, pre=(ILU0, 1), post=(0, 0), use_ms=False)
    assert np.max(np.abs(z.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
