"""Forward substitution of the tiled blocks with the strip in registers (GPU).

Block sizes at the edges of its register shapes (4, 8 and 16 row tiles), with
right-hand sides of one part strip up to several, so that groups hold one to
all of their strips; every element type, factor then solve against the oracle.
Tolerances as in the parity tests: FP64 1e-11, FP32 2e-4 of the largest entry
(kappa <= 10).
"""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev(cuda_ok):
    import torch
    return torch, torch.device("cuda:0")


@pytest.mark.parametrize("dtype", ["complex128", "complex64", "float64", "float32"])
@pytest.mark.parametrize("m,k", [(33, 1), (47, 17), (64, 40), (65, 16), (96, 70), (128, 1),
                                 (129, 17), (208, 40), (256, 3)])
def test_strip_edges(torch_dev, m, k, dtype):
    torch, dev = torch_dev
    from paper_1807_00370_amd.solver import Solver
    print("case strips m=%d k=%d %s" % (m, k, dtype), flush=True)
    dt = getattr(torch, dtype)
    N = 6
    s = (W.random_spd if dtype.startswith("float") else W.random_hpd)(N, m, k, 9300 + m)
    A, B, y = (torch.from_numpy(v).to(dev).to(dt) for v in (s.A, s.B, s.y))
    sol = Solver([N], [m], [k], dtype=dt, device=dev)
    sol.factor(A, B)
    x = sol.solve(y)
    assert torch.equal(sol.factor_solve(A, B, y), x)
    A, B, y = (v.cpu().numpy().astype(np.complex128) for v in (A, B, y))
    xo, io = oracle.solve_cr(A, B, y)
    assert io["status"] == 0 and sol.info_host()[0]["status"] == 0
    tol = 1e-11 if dtype in ("complex128", "float64") else 2e-4
    assert np.abs(x.cpu().numpy() - xo).max() <= tol * np.abs(xo).max()
