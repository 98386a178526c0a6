"""Rows far longer than a grid's (hubs of triangles and tetrahedra, P1 and P2, both models): the element sums on
their own and inside the solver launches against the oracle, and their time, which grows with the simplices
around a row, not with their number times the row's length (needs a GPU)."""
import time

import numpy as np
import pytest
from scipy.spatial import ConvexHull

from helpers import blockerr, dev, host, rel
from oracle import assembly, mobility as mob, pfc as opfc, solve as osolve
import workloads as wl

pytestmark = pytest.mark.gpu
R, M11 = -0.35, 1.0 / opfc.ROS3PW_GAMMA


@pytest.fixture(scope="module")
def pfc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06852_amd import pfc as lib
    return lib


def hub(dim, m, degree=1):
    """Simplices around node 0: m triangles, or the tetrahedra over the hull of m points of a sphere."""
    if dim == 2:
        a = 2.0 * np.pi * np.arange(m) / m
        rim = np.stack([np.cos(a), np.sin(a)], axis=1) * (1.0 + 0.1 * np.sin(3 * a))[:, None]
        faces = np.stack([np.arange(m), (np.arange(m) + 1) % m], axis=1)
    else:
        # a spiral of nearly equal triangles, turned: no tetrahedron is flat
        z = 1.0 - (2.0 * np.arange(m) + 1.0) / m
        phi = np.pi * (1.0 + 5.0 ** 0.5) * np.arange(m) + 0.3
        rim = np.stack([np.sqrt(1.0 - z * z) * np.cos(phi), np.sqrt(1.0 - z * z) * np.sin(phi), z], axis=1)
        faces = np.sort(ConvexHull(rim).simplices, axis=1)
        faces = faces[np.lexsort(faces.T[::-1])]
    xy = np.concatenate([np.zeros((1, dim)), rim])
    nodes = np.concatenate([np.zeros((len(faces), 1), dtype=np.int64), 1 + faces], axis=1).astype(np.int32)
    mesh = wl.Mesh(dim, m + 1, nodes, xy[nodes], 4, 1.0)
    return wl.p2_mesh(mesh) if degree == 2 else mesh


def create(pfc, mesh):
    make = pfc.pfc_mesh_create_p2 if mesh.degree == 2 else pfc.pfc_mesh_create_p1
    return make(mesh.dim, mesh.n, mesh.elem_nodes, mesh.elem_coords)


# the hub's row: 96 entries (the longest whose positions are bytes), 97 and more; the stage right-hand side
# of the mobility model keeps two values per entry in LDS at 96
@pytest.mark.parametrize("dim,m,model", [(2, 16, 1), (2, 95, 1), (2, 96, 1), (2, 200, 1), (3, 60, 1), (3, 130, 1),
                                         (3, 95, 0), (3, 96, 0), (3, 130, 0)])
def test_operators(pfc, dim, m, model):
    mesh = hub(dim, m)
    _operators(pfc, mesh, model, m)


@pytest.mark.parametrize("dim,m", [(2, 5), (3, 12), (3, 24), (3, 40)])  # 3D: hub rows of 55, 115 and 195 entries
def test_operators_p2(pfc, dim, m):
    mesh = hub(dim, m, degree=2)
    _operators(pfc, mesh, 0, m)


def _operators(pfc, mesh, model, seed):
    n = mesh.n
    M, K = assembly.mass_stiffness(mesh)
    rng = np.random.default_rng(seed)
    x = np.concatenate([0.3 * rng.normal(size=n), -0.3 + 0.3 * rng.uniform(-1, 1, n), 0.3 * rng.normal(size=n)])
    y, ys = rng.normal(size=3 * n), 0.1 * rng.normal(size=(3, 3 * n))
    psi, tau = x[n:2 * n], 0.6
    N = assembly.N_matrix(mesh, psi)
    h = create(pfc, mesh)
    inst = pfc.pfc_instance_create(h, pfc.pfc_opts_default(model=model))
    try:
        # sums of at most a few hundred terms of one sign, each with a relative error of a few units in the
        # last place
        Nd, out = dev(np.zeros(M.nnz)), dev(np.zeros(3 * n))
        pfc.pfc_assemble_N(h, dev(psi), Nd)
        assert np.array_equal(N.indices, M.indices)
        assert np.abs(host(Nd) - N.data).max() <= 1e-13 * np.abs(N.data).max()
        xi = x + opfc.ROS3PW_A[(2, 1)] * ys[0]
        prev, c = [ys[0][n:2 * n]], [opfc.ROS3PW_C[(2, 1)]]
        if model:
            ref = mob.apply_AR1(M, K, N, mob.K_plus(mesh, psi), mob.F_mu(mesh, x[:n]), R, tau, M11, y)
            b = mob.stage_rhs_R1(mesh, M, K, R, tau, xi, prev, c)
        else:
            ref = opfc.apply_AR(M, K, N, R, tau, M11, y)
            b = opfc.stage_rhs_R(mesh, M, K, R, tau, xi, prev, c)
        pfc.pfc_apply_AR_x(inst, n, dev(x), R, tau, M11, dev(y), out)
        assert blockerr(host(out), ref) <= 1e-12
        pfc.pfc_stage_rhs(inst, n, dev(x), dev(ys.ravel()), 2, R, tau, out)
        assert blockerr(host(out), b) <= 1e-12
    finally:
        pfc.pfc_instance_destroy(inst)
        pfc.pfc_mesh_destroy(h)


# inside the solver launches: rows of at most 16 entries in rounds of eight, longer ones and P2 in place
@pytest.mark.parametrize("dim,m,degree,model", [(2, 15, 1, 1), (2, 16, 1, 1), (2, 33, 1, 1), (3, 40, 1, 0), (3, 130, 1, 0),
                                                (3, 40, 1, 1), (2, 33, 2, 0), (3, 12, 2, 0), (3, 30, 2, 0)])
def test_step(pfc, dim, m, degree, model):
    mesh = hub(dim, m, degree)
    n = mesh.n
    M, K = assembly.mass_stiffness(mesh)
    tau = 0.01
    psi = -0.3 + 0.05 * np.random.default_rng(m).uniform(-1, 1, n)
    x0 = opfc.consistent_init(mesh, M, K, R, psi)
    run = mob.rosenbrock_run1 if model else osolve.rosenbrock_run
    ref, _ = run(mesh, M, K, x0, R, tau, 1, tol=1e-12)
    h = create(pfc, mesh)
    inst = pfc.pfc_instance_create(h, pfc.pfc_opts_default(outer_tol=1e-12, model=model))
    try:
        x = dev(x0)
        st, _ = pfc.pfc_rosenbrock_run(inst, n, x, R, -0.3, tau, 1, pfc.PFC_INIT_GIVEN)
        assert st == pfc.PFC_OK
        # both stop at a relative residual of 1e-12; the error of a solve is that times its condition
        assert rel(host(x), ref) <= 1e-8
    finally:
        pfc.pfc_instance_destroy(inst)
        pfc.pfc_mesh_destroy(h)


def _best(f):
    import torch
    f()
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


def test_step_time_grows_with_the_simplices(pfc):
    """A step of one Arnoldi step and one inner iteration a solve, which the element sums dominate, on a hub of
    1600 triangles against one of 200: 8 times the simplices and a fixed part; a walk of all simplices for every
    eight entries of the row (64 times the work) measured 46 times the time."""
    t = {}
    for m in (200, 1600):
        mesh = hub(2, m)
        h = create(pfc, mesh)
        inst = pfc.pfc_instance_create(h, pfc.pfc_opts_default(model=1, inner_fixed=[1] * 5, outer_tol=1e6, max_steps=1))
        try:
            psi = -0.3 + 0.05 * np.random.default_rng(m).uniform(-1, 1, mesh.n)
            x = np.concatenate([0.01 * psi, psi, 0.01 * psi])
            t[m] = _best(lambda: pfc.pfc_rosenbrock_run(inst, mesh.n, dev(x), R, -0.3, 1e-3, 1, pfc.PFC_INIT_GIVEN))
        finally:
            pfc.pfc_instance_destroy(inst)
            pfc.pfc_mesh_destroy(h)
    assert t[1600] <= 16 * t[200], t


# N with 16 and 32 lanes of a wave a row (P2, few slices), a thread a row beyond 640 slices, and a last wave that
# is not full; a P2 hub of 46 entries; hub rows of 2048 entries (the most in LDS) and 2049 (in place), also P2
@pytest.mark.parametrize("mesh", [("grid", 2, 3), ("grid", 2, 11), ("grid", 2, 102), ("grid", 3, 3), ("grid", 3, 5),
                                  ("hub", 2, 15, 2), ("hub", 2, 2047, 1), ("hub", 2, 2048, 1), ("hub", 2, 700, 2)],
                         ids=lambda m: "-".join(map(str, m)))
def test_assemble_N(pfc, mesh):
    mesh = hub(*mesh[1:]) if mesh[0] == "hub" else wl.p2_mesh(wl.make_mesh(*mesh[1:], jitter=0.1, seed=71))
    M, _ = assembly.mass_stiffness(mesh)
    psi = -0.3 + 0.3 * np.random.default_rng(71).uniform(-1, 1, mesh.n)
    h = create(pfc, mesh)
    try:
        Nd = dev(np.full(M.nnz, np.nan))
        pfc.pfc_assemble_N(h, dev(psi), Nd)
        ref = assembly.N_matrix(mesh, psi)
        assert np.array_equal(ref.indices, M.indices)
        assert np.abs(host(Nd) - ref.data).max() <= 1e-13 * np.abs(ref.data).max()
    finally:
        pfc.pfc_mesh_destroy(h)


def test_assemble_time_grows_with_the_simplices(pfc):
    """N on a hub of 1600 triangles against one of 200: a walk of all simplices for every 64 entries of the row
    measured 46 times the time; a walk per simplex takes at most 8 times as long."""
    t = {}
    for m in (200, 1600):
        mesh = hub(2, m)
        h = create(pfc, mesh)
        try:
            psi, N = dev(np.full(mesh.n, -0.3)), dev(np.zeros(7 * m + 1))
            N = N[:pfc.pfc_mesh_export_csr(h)[1].size]
            t[m] = _best(lambda: [pfc.pfc_assemble_N(h, psi, N) for _ in range(5)])
        finally:
            pfc.pfc_mesh_destroy(h)
    assert t[1600] <= 14 * t[200], t
