"""Blocks of 1..8, several per wave (GPU): every block size, odd block counts
(a last wave with fewer blocks), right-hand sides below, at and beyond the
columns one pass covers, every element type; one-sided and with the Algorithm
1 tail; factor then solve equals the fused call bit for bit.  Tolerances as in
the parity tests (kappa <= 10)."""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 3), (70, 1), (131, 5), (64, 9), (33, 17), (40, 41)]


@pytest.fixture(scope="module")
def torch_dev(cuda_ok):
    import torch
    return torch, torch.device("cuda:0")


@pytest.mark.parametrize("dtype", ["complex128", "complex64", "float64", "float32"])
@pytest.mark.parametrize("m", range(1, 9))
def test_small_blocks(torch_dev, m, dtype):
    torch, dev = torch_dev
    from paper_1807_00370_amd.solver import Solver
    dt = getattr(torch, dtype)
    gen = W.random_spd if dtype.startswith("float") else W.random_hpd
    tol = 1e-11 if dtype in ("complex128", "float64") else 2e-4
    for N, k in SHAPES:
        print("case small m=%d N=%d k=%d %s" % (m, N, k, dtype), flush=True)
        s = gen(N, m, k, 9300 + 10 * N + m)
        A, B, y = (torch.from_numpy(np.ascontiguousarray(v)).to(dev).to(dt)
                   for v in (s.A, s.B, s.y))
        xo, io = oracle.solve_cr(*(v.cpu().numpy().astype(np.complex128) for v in (A, B, y)))
        assert io["status"] == 0
        for tail in (0, None):
            sol = Solver([N], [m], [k], dtype=dt, device=dev, pcr_tail_blocks=tail)
            x = sol.factor_solve(A, B, y)
            sol.factor(A, B)
            assert torch.equal(sol.solve(y), x)
            assert sol.info_host()[0]["status"] == 0
            assert np.abs(x.cpu().numpy() - xo).max() <= tol * np.abs(xo).max()


def test_small_blocks_mixed_batch(torch_dev):
    """Waves whose blocks belong to different systems (sizes 1..8 in one
    batch), one of them indefinite: its neighbours are untouched."""
    torch, dev = torch_dev
    from paper_1807_00370_amd.solver import Solver
    shapes = [(5 + 3 * i, 1 + i % 8, 1 + i % 11) for i in range(24)]
    systems = [W.random_hpd(N, m, k, 9500 + i, shift_scale=2.0 if i == 7 else 0.0)
               for i, (N, m, k) in enumerate(shapes)]
    A, B, y = (torch.from_numpy(np.concatenate([getattr(s, q).ravel() for s in systems])).to(dev)
               for q in "ABy")
    sol = Solver([s.N for s in systems], [s.m for s in systems], [s.k for s in systems], device=dev)
    x, off = sol.factor_solve(A, B, y).cpu().numpy(), 0
    rec = sol.info_host()
    for i, s in enumerate(systems):
        xo, io = oracle.solve_cr(s.A, s.B, s.y)
        xi = x[off:off + s.y.size].reshape(s.y.shape)
        off += s.y.size
        assert rec["status"][i] == io["status"] == (1 if i == 7 else 0)
        if i == 7:
            assert np.isnan(xi).all()
        else:
            assert np.abs(xi - xo).max() <= 1e-11 * np.abs(xo).max()
