"""Heat applies in every work unit that heat_apply chooses between beyond the
overlapping tiles (which take meshes of up to 2048 tiles, one per 3 cells and
direction): bricks, and slabs of one, two and four sub-bricks along x, with and
without empty and clipped sub-bricks, in each form of the operator.

Rows of the operator from the oracle's cell matrices: whole lines of nodes
along x, y and z through the corners, across the planes between bricks and
slabs and through the middle, and 600 random nodes; every entry of y has to be
written.  Bars as in test_gpu_heat.py, 1e-12 (FP64) and 2e-6 (FP32), relative to
the largest entry.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2501_18781_amd import mf
from paper_2501_18781_amd import workloads as W

pytestmark = pytest.mark.gpu


def tiles(n):
    return int(np.prod([1 if c <= 4 else (c + 1) // 3 for c in n]))


def sampled_rows(mesh):
    N = [2 * c + 1 for c in mesh.n]
    id_ = lambda i, j, k: i + N[0] * (j + N[1] * k)
    cuts = [sorted({0, 7, 8, 9, 32, N[d] // 2, N[d] - 2, N[d] - 1} & set(range(N[d]))) for d in range(3)]
    rows = [np.random.default_rng(1).integers(0, mesh.n_nodes, 600)]
    for a, b, c in ((0, 1, 2), (1, 0, 2), (2, 0, 1)):  # lines along a
        for u, v in zip(cuts[b], reversed(cuts[c])):
            ijk = [None, None, None]
            ijk[a], ijk[b], ijk[c] = np.arange(N[a]), u, v
            rows.append(id_(*ijk))
    return np.unique(np.concatenate([np.atleast_1d(r) for r in rows]))


def dev(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda").to(dtype)


def check(n, form, precision=mf.MF_FP64, equal_edges=True, dirichlet=W.FACE_XLO | W.FACE_YHI | W.FACE_ZLO):
    """form: words of linear, sine, points, conv, transpose, melt."""
    f32 = precision == mf.MF_FP32
    dtype, tol = (torch.float32, 2e-6) if f32 else (torch.float64, 1e-12)
    print(f"slab shapes n={n} {form} fp32={f32} equal={equal_edges}", flush=True)
    words = form.split()
    mesh = W.Mesh(n, hi=tuple(c / max(n) for c in n) if equal_edges else (1.0, 1.0, 1.0), dirichlet=dirichlet)
    eps = 2.0 * max(mesh.h)
    melt = "melt" in words
    p = W.HeatParams(heaviside=int("sine" in words), eps=eps if "sine" in words else 0.0, penalty=2.0e9 if melt else 0.0)
    rnd = lambda a: a.astype(np.float32).astype(np.float64) if f32 else a  # what the call is given
    phi = rnd(W.phi_sphere(mesh, 0.3, eps))
    x = rnd(W.uniform(4, mesh.n_nodes))
    ctx = mf.Context(mesh)
    kw = {}
    if "points" in words:
        g = np.random.default_rng(6)
        kq, rcq = rnd(g.uniform(0.3, 30.0, mesh.n_cells * 27)), rnd(g.uniform(5e3, 5e6, mesh.n_cells * 27))
        op = mf.heat_operator(ctx, p, k_q=dev(kq, dtype), rc_q=dev(rcq, dtype), precision=precision)
        kw = {"kq": kq, "rcq": rcq}
    else:
        kw["phi"] = phi
        u0 = W.taylor_green(mesh) if "conv" in words else None
        Tc = 1800.0 + 600.0 * W.uniform(8, mesh.n_nodes) if melt else None
        op = mf.heat_operator(ctx, p, phi=dev(phi, dtype), precision=precision,
                              u0=None if u0 is None else dev(u0, dtype).reshape(-1),
                              T_coef=None if Tc is None else dev(Tc, dtype))
        if u0 is not None:
            kw["u0"] = u0
        if Tc is not None:
            kw["Tc"] = Tc
    xd = dev(x, dtype)
    rows = sampled_rows(mesh)
    at = torch.as_tensor(rows, device="cuda")
    for transpose in ([False, True] if "conv" in words else [False]):
        y = torch.full_like(xd, float("nan"))
        (mf.operator_apply_transpose if transpose else mf.operator_apply)(op, xd, y)
        assert not torch.isnan(y).any()
        ref = O.heat_rows(mesh, p, x, rows, transpose=transpose, **kw)
        err = np.abs(y[at].cpu().double().numpy() - ref).max() / np.abs(ref).max()
        assert err <= tol, (transpose, err)


# FP32.  Sub-bricks along x, slots of the slabs: 10 of 10 and 5 of 6 and 11 of 12
# in pairs (the last sub-brick empty), 2 of 2; one and three bricks along x, and
# the sine form up to 1024 bricks: slabs of one; 13824 bricks, 13248 with 23 of 24
# slots and 10164 with 21 of 24: slabs of four
FP32 = [((39, 41, 43), "linear", True), ((18, 61, 70), "linear", False), ((42, 45, 41), "sine", True),
        ((41, 43, 42), "points", True), ((7, 98, 97), "sine", False), ((4, 150, 146), "points", False),
        ((11, 77, 83), "linear", False), ((38, 40, 39), "sine", True), ((93, 95, 94), "linear", True),
        ((90, 94, 95), "sine", False), ((82, 87, 86), "points", True)]


@pytest.mark.parametrize("n,form,equal", FP32)
def test_fp32(gpu, n, form, equal):
    assert tiles(n) > 2048
    check(n, form, mf.MF_FP32, equal)


# FP64.  Bricks: three phases, the convective form and, on large meshes, its
# transpose; slabs of one; slabs of four in which one to three sub-bricks are
# empty: 11 of 12 slots (1320 bricks), 13 of 16 (13728), 22 of 24 (13200), 18 of 20
# (6840), 9 of 12 (7308), 21 of 24 (10164; its transpose bricks), 23 of 24 (11132,
# 13248), 19 of 20 (7220)
BRICK = [((38, 41, 35), "melt", False), ((45, 50, 51), "conv", True), ((45, 50, 51), "conv sine", False),
         ((35, 129, 131), "conv", False)]
ONE = [((42, 58, 47), "linear", False), ((50, 37, 61), "sine", False), ((41, 42, 43), "points", True),
       ((45, 41, 39), "conv", True), ((45, 41, 39), "conv sine", False), ((38, 41, 35), "melt sine", True)]
FOUR = [((43, 47, 39), "linear", True), ((50, 127, 129), "linear", False), ((86, 98, 95), "sine", True),
        ((69, 75, 78), "points", False), ((35, 111, 113), "points", True), ((83, 86, 87), "conv", False),
        ((90, 86, 87), "conv", True), ((91, 95, 96), "conv sine", True), ((73, 76, 79), "melt", True),
        ((91, 95, 96), "melt sine", False)]


@pytest.mark.parametrize("n,form,equal", BRICK + ONE + FOUR)
def test_fp64(gpu, n, form, equal):
    assert tiles(n) > 2048
    check(n, form, mf.MF_FP64, equal)
