"""Blocks whose last 16 x 16 tile is partial (GPU): the tile Cholesky leaves out
the panels of four columns past the block's edge, and a launch deals a block's
strips over several waves.  Every panel edge of one and two tiles against the
oracle, a bad pivot in every column, and the same bits however many waves share
a block.  Tolerances as in the parity tests: FP64 1e-11, FP32 2e-4 of the
largest entry (kappa <= 10).
"""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["complex128", "complex64", "float64", "float32"])
@pytest.mark.parametrize("m", [10, 12, 13, 18, 20, 21, 25, 28, 29, 36, 37, 44])
def test_panel_edges(cuda_ok, m, dtype):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case panel m=%d %s" % (m, dtype), flush=True)
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    s = (W.random_spd if dtype.startswith("float") else W.random_hpd)(21, m, 5, 9700 + m)
    A, B, y = (torch.from_numpy(v).to(dev).to(dt) for v in (s.A, s.B, s.y))
    sol = Solver([21], [m], [5], dtype=dt, device=dev)
    x = sol.factor_solve(A, B, y)
    sol.factor(A, B)
    assert torch.equal(sol.solve(y), x)
    xo, io = oracle.solve_cr(*(v.cpu().numpy().astype(np.complex128) for v in (A, B, y)))
    assert io["status"] == 0 and sol.info_host()[0]["status"] == 0
    tol = 1e-11 if dtype in ("complex128", "float64") else 2e-4
    assert np.abs(x.cpu().numpy() - xo).max() <= tol * np.abs(xo).max()


@pytest.mark.parametrize("m", [13, 21, 28, 29])
def test_bad_pivot_in_partial_tile(cuda_ok, m):
    import torch
    from paper_1807_00370_amd.solver import Solver
    dev = torch.device("cuda:0")
    A = np.tile(2.0 * np.eye(m, dtype=np.complex128), (m + 1, 1, 1))
    A[np.arange(m), np.arange(m), np.arange(m)] = -1.0
    n = m + 1
    sol = Solver([1] * n, [m] * n, [1] * n, device=dev)
    sol.check_hpd(torch.from_numpy(A.ravel()).to(dev), torch.empty(0, dtype=torch.complex128, device=dev))
    rec = sol.info_host()
    assert (rec["status"] == np.r_[np.ones(m), 0]).all()
    assert (rec["level"][:m] == 0).all() and (rec["block"][:m] == 1).all()


@pytest.mark.parametrize("N,m,k", [(600, 20, 40), (300, 9, 17), (513, 32, 1), (705, 17, 33)])
def test_same_bits_for_any_split(cuda_ok, N, m, k):
    """How many waves share a block does not change a bit of x."""
    import torch
    from paper_1807_00370_amd.solver import Solver
    dev = torch.device("cuda:0")
    s = W.random_hpd(N, m, k, 9800 + m)
    A, B, y = (torch.from_numpy(v).to(dev) for v in (s.A, s.B, s.y))
    sol = Solver([N], [m], [k], device=dev, schedule="pcr")
    x = sol.factor_solve(A, B, y).clone()
    assert sol.info_host()[0]["status"] == 0
    for waves in (1, 1024, 4 * N, 1 << 20):
        sol.plan.set_tuning("tw=%d;" % waves)
        assert torch.equal(sol.factor_solve(A, B, y), x)
