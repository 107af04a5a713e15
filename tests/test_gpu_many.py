"""Launches of many blocks (GPU).

* Real data gives the same bits as complex data with zero imaginary parts, also
  above 128 and with more than 256 blocks in a launch.
* FP64 complex blocks above 128, imaginary parts and partial tiles included, with
  more than 256 of them in a launch: a batch of copies of a few systems, each
  copy the same bits as its system alone, and the oracle's solution.
* Blocks of 1..4 in FP64 with so many waves that work-groups hold four.

Tolerance as in the parity tests: 1e-11 of the largest entry (kappa <= 10).
"""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,m,k", [(516, 130, 3), (600, 144, 17), (520, 256, 1), (600, 96, 2)])
def test_real_equals_complex_many_blocks(cuda_ok, N, m, k):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case real-complex N=%d m=%d k=%d" % (N, m, k), flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(9000 + m)
    B = torch.randn(N - 1, m, m, dtype=torch.float64, device=dev, generator=g) * (0.3 / m ** 0.5)
    M = torch.randn(N, m, m, dtype=torch.float64, device=dev, generator=g)
    A = M @ M.mT.contiguous() / m
    A = (A + A.mT) / 2 + 3.0 * torch.eye(m, dtype=torch.float64, device=dev)
    y = torch.randn(N, m, k, dtype=torch.float64, device=dev, generator=g)
    x = Solver([N], [m], [k], dtype=torch.float64, device=dev).factor_solve(A, B, y)
    sol = Solver([N], [m], [k], dtype=torch.complex128, device=dev)
    xc = sol.factor_solve(*(v.to(torch.complex128) for v in (A, B, y)))
    assert sol.info_host()[0]["status"] == 0
    assert torch.equal(xc.real, x) and bool((xc.imag == 0).all())
    r = A @ x - y
    r[1:] += B @ x[:-1]
    r[:-1] += B.mT.contiguous() @ x[1:]
    assert float(r.norm() / y.norm()) <= 1e-12


@pytest.mark.parametrize("m,k", [(129, 17), (144, 33), (200, 7), (256, 1)])
def test_wide_complex_blocks_in_one_launch(cuda_ok, m, k):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case wide m=%d k=%d" % (m, k), flush=True)
    dev, N, copies = torch.device("cuda:0"), 3, 130
    base = [W.random_hpd(N, m, k, 9400 + m + i) for i in range(2)]
    n = copies * len(base)  # N // 2 + 1 eliminated blocks each at the first level

    def all_of(q):
        return torch.from_numpy(np.concatenate([getattr(s, q).ravel() for s in base])).to(dev).repeat(copies)

    sol = Solver([N] * n, [m] * n, [k] * n, device=dev)
    A, B, y = (all_of(q) for q in "ABy")
    x = sol.factor_solve(A, B, y).clone()
    assert (sol.info_host()["status"] == 0).all()
    sol.factor(A, B)
    assert torch.equal(sol.solve(y), x)
    x = x.reshape(copies, len(base), N, m, k)
    for i, s in enumerate(base):
        a, b, c = (torch.from_numpy(getattr(s, q)).to(dev) for q in "ABy")
        alone = Solver([N], [m], [k], device=dev).factor_solve(a, b, c)
        assert torch.equal(x[:, i], alone.expand(copies, -1, -1, -1))
        xo, io = oracle.solve_cr(s.A, s.B, s.y)
        assert io["status"] == 0
        assert np.abs(alone.cpu().numpy() - xo).max() <= 1e-11 * np.abs(xo).max()


@pytest.mark.parametrize("dtype", ["complex128", "float64"])
@pytest.mark.parametrize("N,m,k", [(17001, 3, 2), (16400, 4, 1), (20000, 1, 5), (9001, 8, 1)])
def test_many_small_blocks(cuda_ok, N, m, k, dtype):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case many small N=%d m=%d k=%d %s" % (N, m, k, dtype), flush=True)
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    s = (W.random_spd if dtype == "float64" else W.random_hpd)(N, m, k, 9450 + m)
    A, B, y = (torch.from_numpy(v).to(dev).to(dt) for v in (s.A, s.B, s.y))
    sol = Solver([N], [m], [k], dtype=dt, device=dev)
    x = sol.factor_solve(A, B, y)
    sol.factor(A, B)
    assert torch.equal(sol.solve(y), x)
    xo, io = oracle.solve_cr(s.A, s.B, s.y)
    assert io["status"] == 0 and sol.info_host()[0]["status"] == 0
    assert np.abs(x.cpu().numpy() - xo).max() <= 1e-11 * np.abs(xo).max()
