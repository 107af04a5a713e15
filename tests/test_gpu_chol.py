"""Tiled Cholesky held in registers (GPU): a bad pivot at the edges of every
tile is reported for its own system alone, for every element type and at the
edges of the kernel's register shapes (4, 8 and 16 tile columns)."""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["complex128", "complex64", "float64", "float32"])
@pytest.mark.parametrize("m", [33, 64, 65, 113, 128, 129, 256])
def test_bad_pivot_in_every_tile(cuda_ok, m, dtype):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case pivot m=%d %s" % (m, dtype), flush=True)
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    cols = sorted({c for c in range(m) if c % 16 in (0, 15)} | {m - 1})
    s = (W.random_spd if dtype.startswith("float") else W.random_hpd)(1, m, 1, 9500 + m)
    A = np.tile(s.A, (len(cols) + 1, 1, 1))
    for i, c in enumerate(cols):
        A[i, c, c] = -1.0
    n = len(A)
    sol = Solver([1] * n, [m] * n, [1] * n, dtype=dt, device=dev)
    y = np.tile(s.y, (n, 1, 1))
    x = sol.factor_solve(torch.from_numpy(A).to(dev).to(dt), torch.empty(0, dtype=dt, device=dev),
                         torch.from_numpy(y).to(dev).to(dt))
    rec = sol.info_host()
    assert (rec["status"] == np.r_[np.ones(n - 1), 0]).all()
    assert (rec["level"][:-1] == 0).all() and (rec["block"][:-1] == 1).all()
    xo, io = oracle.solve_cr(s.A, s.B, s.y)
    tol = 1e-11 if dtype in ("complex128", "float64") else 2e-4
    assert np.abs(x.cpu().numpy().reshape(n, m, 1)[-1] - xo[0]).max() <= tol * np.abs(xo).max()
