"""Stored-factor solves with few right-hand-side strips in single precision
(GPU): a work-group per strip and a wave per row tile, at the edges of tiles and
strips, on both sides of the launch rule and with blocks of different sizes in
one launch.  The same bits as the fused call, and against the oracle (2e-4 of
the largest entry, as in the parity tests; kappa <= 10).
"""
import numpy as np
import pytest

import oracle
from paper_1807_00370_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(systems, dtype):
    import torch
    from paper_1807_00370_amd.solver import Solver
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    A, B, y = (torch.from_numpy(np.concatenate([getattr(s, q).ravel() for s in systems])).to(dev).to(dt)
               for q in "ABy")
    sol = Solver([s.N for s in systems], [s.m for s in systems], [s.k for s in systems], dtype=dt,
                 device=dev)
    fused = sol.factor_solve(A, B, y).clone()
    sol.factor(A, B)
    x = sol.solve(y)
    assert torch.equal(x, fused)
    x, off = x.cpu().numpy(), 0
    assert (sol.info_host()["status"] == 0).all()
    for s in systems:
        a, b, c = (np.asarray(v).astype(dtype).astype(np.complex128) for v in (s.A, s.B, s.y))
        xo, io = oracle.solve_cr(a, b, c)
        xi = x[off:off + s.y.size].reshape(s.y.shape)
        off += s.y.size
        assert np.abs(xi - xo).max() <= 2e-4 * np.abs(xo).max()


@pytest.mark.parametrize("dtype", ["complex64", "float32"])
@pytest.mark.parametrize("N,m,k", [(5, 65, 1), (6, 80, 16), (3, 127, 17), (4, 144, 33), (2, 241, 1),
                                   (3, 256, 48), (600, 66, 97)])
def test_few_strips(cuda_ok, N, m, k, dtype):
    print("case few N=%d m=%d k=%d %s" % (N, m, k, dtype), flush=True)
    gen = W.random_spd if dtype.startswith("float") else W.random_hpd
    _run([gen(N, m, k, 9600 + m)], dtype)


@pytest.mark.parametrize("dtype", ["complex64", "float32"])
def test_few_strips_mixed_sizes(cuda_ok, dtype):
    gen = W.random_spd if dtype.startswith("float") else W.random_hpd
    _run([gen(N, m, k, 9650 + m) for N, m, k in ((3, 66, 1), (4, 250, 5), (2, 128, 20), (5, 97, 2))],
         dtype)
