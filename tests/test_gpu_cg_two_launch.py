"""CG on meshes of one-brick slabs (two launches per iteration): the iterates
after 1, 5 and 9 steps (9: x is completed after the first poll of the state)
against the FP64 oracle's, with clipped bricks, walls on some faces, a single
brick, and each way the coefficients are given.

Bar: 1e-10 normwise.  An iterate's rounding error is that of a sum over the
nodes (below 1e-13 relative for these sizes) per step, amplified by at most the
spread of the Jacobi-scaled spectrum (below 100 for these operators).
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2501_18781_amd import mf
from paper_2501_18781_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("n,dirichlet,hi,hkind,points,jacobi", [
    ((4, 4, 4), 0, (1.0, 1.0, 1.0), 0, False, True),
    ((3, 9, 5), W.ALL_FACES, (0.4, 1.0, 0.6), 1, False, True),
    ((8, 5, 13), W.FACE_XLO | W.FACE_YHI, (1.0, 1.0, 1.0), 0, True, False),
    ((13, 12, 8), W.FACE_ZHI | W.FACE_XHI, (1.0, 1.0, 1.0), 0, False, False),
    ((18, 16, 15), W.ALL_FACES, (18 / 16, 1.0, 15 / 16), 1, True, True),
])
def test_iterates(gpu, n, dirichlet, hi, hkind, points, jacobi):
    print(f"two-launch CG n={n} dirichlet={dirichlet} H={hkind} points={points} jacobi={jacobi}", flush=True)
    mesh = W.Mesh(n, hi=hi, dirichlet=dirichlet)
    eps = 2.0 / max(n)
    p = W.HeatParams(heaviside=hkind, eps=eps if hkind else 0.0)
    phi = W.phi_sphere(mesh, 0.3, eps)
    ctx = mf.Context(mesh)
    if points:
        kq, rcq = O.heat_qp_coeffs(mesh, p, phi)
        A = O.heat_matrix(mesh, p, kq=kq, rcq=rcq)
        op = mf.heat_operator(ctx, p, k_q=dev(kq).reshape(-1), rc_q=dev(rcq).reshape(-1))
    else:
        A = O.heat_matrix(mesh, p, phi=phi)
        op = mf.heat_operator(ctx, p, phi=dev(phi))
    b = A @ W.uniform(3, mesh.n_nodes)
    dinv = None if jacobi else np.ones(mesh.n_nodes)
    for k in (1, 5, 9):
        ref = O.jacobi_cg(A, b, 0.0, k, dinv=dinv).x
        x = torch.full((mesh.n_nodes,), float("nan"), dtype=torch.float64, device="cuda")
        info = mf.cg_solve(op, dev(b), x, 0.0, k, precond=mf.MF_PC_JACOBI if jacobi else mf.MF_PC_NONE)
        assert info.status == mf.MF_NOT_CONVERGED and info.iters == k
        assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref), k
