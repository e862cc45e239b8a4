"""Heat applies in overlapping tiles (small meshes, one launch) against the FP64
oracle: one tile, one tile and a bit, clipped last tiles, more tiles than SIMDs,
in every form of the operator.

Bars as in test_gpu_heat.py: 1e-12 (FP64) and 2e-6 (FP32), normwise and
element-wise.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2501_18781_amd import mf
from paper_2501_18781_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL64, TOL32 = 1e-12, 2e-6


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def relerr(a, b):
    d = a.cpu().double().numpy() - b
    return max(np.linalg.norm(d) / np.linalg.norm(b), np.abs(d).max() / np.abs(b).max())


def apply(op, x, transpose=False):
    y = torch.full_like(x, float("nan"))  # every entry has to be written
    (mf.operator_apply_transpose if transpose else mf.operator_apply)(op, x, y)
    return y


SIZES = [((4, 5, 7), W.ALL_FACES), ((8, 10, 11), W.FACE_XLO | W.FACE_YHI), ((13, 1, 2), W.FACE_XHI | W.FACE_ZLO),
         ((3, 6, 9), 0), ((37, 31, 36), W.FACE_ZHI | W.FACE_YLO)]


@pytest.mark.parametrize("n,dirichlet", SIZES)
def test_every_form(gpu, n, dirichlet):
    print(f"tiles n={n} dirichlet={dirichlet}", flush=True)
    mesh = W.Mesh(n, dirichlet=dirichlet)
    eps = 2.0 / max(n)
    p = W.HeatParams()
    phi = W.phi_sphere(mesh, 0.3, eps)
    x = W.uniform(7, mesh.n_nodes)
    x32 = x.astype(np.float32)
    u0 = np.stack([W.uniform(8 + c, mesh.n_nodes) for c in range(3)])
    ctx = mf.Context(mesh)
    A = O.heat_matrix(mesh, p, phi=phi)
    assert relerr(apply(mf.heat_operator(ctx, p, phi=dev(phi)), dev(x)), A @ x) <= TOL64
    op = mf.heat_operator(ctx, p, phi=dev(phi, torch.float32), precision=mf.MF_FP32)
    assert relerr(apply(op, dev(x32, torch.float32)), A @ x32.astype(np.float64)) <= TOL32
    kq, rcq = O.heat_qp_coeffs(mesh, p, phi)
    op = mf.heat_operator(ctx, p, k_q=dev(kq).reshape(-1), rc_q=dev(rcq).reshape(-1))
    assert relerr(apply(op, dev(x)), A @ x) <= TOL64
    B = O.heat_matrix(mesh, p, phi=phi, u0=u0)
    op = mf.heat_operator(ctx, p, phi=dev(phi), u0=dev(u0).reshape(-1))
    assert relerr(apply(op, dev(x)), B @ x) <= TOL64
    assert relerr(apply(op, dev(x), transpose=True), B.T @ x) <= TOL64
