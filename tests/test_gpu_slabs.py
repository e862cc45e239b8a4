"""Heat applies on meshes large enough for the four-wavefront slabs, clipped in
every direction, against the FP64 oracle.

Bars as in test_gpu_heat.py: 1e-12 (FP64) and 2e-6 (FP32), normwise and
element-wise; CG iterations within 1 of the oracle's.
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


def case(n, dirichlet, hkind=0):
    mesh = W.Mesh(n, dirichlet=dirichlet)
    eps = 2.0 / max(n)
    return mesh, W.HeatParams(heaviside=hkind, eps=eps if hkind else 0.0), W.phi_sphere(mesh, 0.3, eps)


def apply(op, x, transpose=False):
    y = torch.full_like(x, float("nan"))  # every entry has to be written
    (mf.operator_apply_transpose if transpose else mf.operator_apply)(op, x, y)
    return y


# sub-bricks along x: 9 of 12 (three of four used, the least a slab takes) and
# 12 of 12 with the last one clipped to a single cell
@pytest.mark.parametrize("n,dirichlet", [((36, 61, 47), W.FACE_XLO | W.FACE_YHI | W.FACE_ZLO), ((45, 50, 41), 0),
                                         ((45, 41, 50), W.ALL_FACES)])
def test_plain_apply_and_cg(gpu, n, dirichlet):
    print(f"slab apply n={n} dirichlet={dirichlet}", flush=True)
    mesh, p, phi = case(n, dirichlet)
    A = O.heat_matrix(mesh, p, phi=phi)
    x = W.uniform(0, mesh.n_nodes)
    ref = A @ x
    ctx = mf.Context(mesh)
    op = mf.heat_operator(ctx, p, phi=dev(phi))
    assert relerr(apply(op, dev(x)), ref) <= TOL64
    xf = x.astype(np.float32)
    opf = mf.heat_operator(ctx, p, phi=dev(phi, torch.float32), precision=mf.MF_FP32)
    assert relerr(apply(opf, dev(xf, torch.float32)), A @ xf.astype(np.float64)) <= TOL32
    sol = O.jacobi_cg(A, ref, 1e-10)
    xs = torch.empty_like(dev(x))
    info = mf.cg_solve(op, dev(ref), xs, 1e-10, 500)
    assert info.converged and abs(info.iters - sol.iters) <= 1 and info.rel_res <= 1.5e-10


def test_heavy_forms(gpu):
    n, dirichlet = (61, 58, 62), W.FACE_XHI | W.FACE_YLO | W.FACE_ZHI
    print(f"slab apply, sine Heaviside, convection, coefficients per point n={n}", flush=True)
    mesh, p, phi = case(n, dirichlet, hkind=1)
    x = W.uniform(1, mesh.n_nodes)
    ctx = mf.Context(mesh)
    A = O.heat_matrix(mesh, p, phi=phi)
    op = mf.heat_operator(ctx, p, phi=dev(phi))
    assert relerr(apply(op, dev(x)), A @ x) <= TOL64
    kq = torch.empty(mesh.n_cells * 27, dtype=torch.float64, device="cuda")
    rcq = torch.empty_like(kq)
    mf.heat_qp_coeffs(op, kq, rcq)
    assert relerr(apply(mf.heat_operator(ctx, p, k_q=kq, rc_q=rcq), dev(x)), A @ x) <= TOL64
    del A
    u0 = W.taylor_green(mesh)
    C = O.heat_matrix(mesh, p, phi=phi, u0=u0)
    op = mf.heat_operator(ctx, p, phi=dev(phi), u0=dev(u0))
    assert relerr(apply(op, dev(x)), C @ x) <= TOL64
    assert relerr(apply(op, dev(x), transpose=True), C.T @ x) <= TOL64
