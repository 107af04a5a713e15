"""Right-hand-side columns of blocks of 1..8 dealt over several waves (GPU):
column counts at the edges of a wave's share, against the oracle, and every
column the same bits as when it is solved alone; factored beforehand or in one
pass.  Tolerances as in the parity tests: FP64 1e-11, FP32 2e-4 of the largest
entry (kappa <= 10).
"""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["complex128", "complex64", "float64"])
@pytest.mark.parametrize("N,m,k", [(1, 1, 65), (2, 3, 17), (40, 4, 129), (33, 8, 33), (21, 5, 300),
                                   (700, 2, 70), (700, 8, 40), (5000, 7, 41)])
def test_columns_over_waves(cuda_ok, N, m, k, dtype):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case columns N=%d m=%d k=%d %s" % (N, m, k, dtype), flush=True)
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    s = (W.random_spd if dtype.startswith("float") else W.random_hpd)(N, m, k, 9900 + m)
    A, B, y = (torch.from_numpy(np.ascontiguousarray(v)).to(dev).to(dt) for v in (s.A, s.B, s.y))
    sol = Solver([N], [m], [k], dtype=dt, device=dev)
    x = sol.factor_solve(A, B, y)
    sol.factor(A, B)
    assert torch.equal(sol.solve(y), x)
    one = Solver([N], [m], [1], dtype=dt, device=dev)
    one.factor(A, B)
    for c in sorted({0, m - 1, m, min(k - 1, 8), k // 2, k - 1}):
        assert torch.equal(one.solve(y[:, :, c:c + 1].contiguous()), x[:, :, c:c + 1])
    xo, io = oracle.solve_cr(*(v.cpu().numpy().astype(np.complex128) for v in (A, B, y)))
    assert io["status"] == 0 and sol.info_host()[0]["status"] == 0
    tol = 1e-11 if dtype in ("complex128", "float64") else 2e-4
    assert np.abs(x.cpu().numpy() - xo).max() <= tol * np.abs(xo).max()
