"""CG in two launches per iteration: where the host polls the solver's state is
no part of what is computed.

Iteration 16 ends the solve in both runs (maxit).  With rtol = 0 a poll follows
it and the poll's own test reads the residual; with rtol = 1e-100 (the same
iterates: neither tolerance is met) the second batch is 16 iterations long, no
poll falls there and the apply's test reads it.  Both sum the same partials, so
the reported residual estimate has to be the same number, and x too.
"""
import numpy as np
import pytest
import torch

from paper_2501_18781_amd import mf
from paper_2501_18781_amd import workloads as W

pytestmark = pytest.mark.gpu


# 60, 216, 504 and 512 partials per sum: one load per lane, several, and a whole pass
@pytest.mark.parametrize("n", [(15, 17, 9), (24, 23, 21), (32, 36, 25), (33, 36, 35)])
def test_residual_does_not_depend_on_the_poll(gpu, n):
    print(f"CG poll n={n}", flush=True)
    mesh = W.Mesh(n, dirichlet=W.FACE_XLO | W.FACE_ZHI)
    phi = torch.as_tensor(W.phi_sphere(mesh, 0.3, 2.0 / max(n)), dtype=torch.float64, device="cuda")
    op = mf.heat_operator(mf.Context(mesh), W.HeatParams(dt=1.0), phi=phi)
    for seed in range(8):  # a difference in the last bits may vanish in the square root
        b = torch.as_tensor(W.uniform(seed, mesh.n_nodes), dtype=torch.float64, device="cuda")
        x0, x1 = torch.empty_like(b), torch.empty_like(b)
        i0 = mf.cg_solve(op, b, x0, 0.0, 16)
        i1 = mf.cg_solve(op, b, x1, 1e-100, 16)
        assert i0.iters == i1.iters == 16
        assert i0.rel_res_est == i1.rel_res_est, seed
        assert torch.equal(x0, x1)
