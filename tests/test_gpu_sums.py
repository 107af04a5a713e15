"""Rounding order of the 16 x 16 tile Cholesky (GPU, blocks of 9..32).

A = I + c E, c = 2^-27 off the diagonal (times a unit phase): every product
of two entries of a row of L is 2^-54 to first order, half a unit in the last
place below 1, so a sum that starts from the diagonal entry rounds each of
them away, one that starts from zero keeps them all.  The last diagonal entry
of A^-1 is 1 / (1 - (m - 1) c^2) = 1 + (m - 1) / 4 units of 2^-52 (the next
term, from c^3, is below 2^-72).  It is the square of the last inverse pivot.

Tolerance, in units of 2^-52: the pivot's own rounding 0.25, up to three
products in the pivot's panel of four columns 0.75, the inverse square root
twice 1, the two products 0.5: 2.5, below the (m - 1) / 4 >= 3.75 that sums
from the diagonal lose.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,phase", [("complex128", 1.0), ("complex128", 1j), ("float64", 1.0)])
@pytest.mark.parametrize("m", [16, 17, 24, 32])
def test_products_are_summed_before_the_diagonal(cuda_ok, m, dtype, phase):
    import torch
    from paper_1807_00370_amd.solver import Solver
    print("case sums m=%d %s" % (m, dtype), flush=True)
    dev, dt = torch.device("cuda:0"), getattr(torch, dtype)
    low = np.tril(np.full((m, m), 2.0 ** -27 * phase), -1)
    A = torch.from_numpy((np.eye(m) + low + low.conj().T)[None].astype(dtype)).to(dev)
    y = torch.zeros(1, m, 1, dtype=dt, device=dev)
    y[0, m - 1, 0] = 1
    sol = Solver([1], [m], [1], dtype=dt, device=dev)
    x = sol.factor_solve(A, torch.empty(0, dtype=dt, device=dev), y)[0, m - 1, 0].item()
    assert sol.info_host()[0]["status"] == 0
    assert abs((x.real - 1.0) * 2.0 ** 52 - (m - 1) / 4) <= 2.5
