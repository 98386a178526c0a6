"""Element sums formed row by row (N(psi), the cubic load, the operator apply and the stage
right-hand side) at the row lengths where their launch changes: rows staged whole in LDS (up to 96
entries), longer rows summed in rounds, and a last slice that is not full (needs a GPU)."""
import numpy as np
import pytest

from helpers import blockerr, dev, host
from oracle import assembly, pfc as opfc, solve as osolve
import workloads as wl

pytestmark = pytest.mark.gpu


def wheel(m, degree=1):
    """m triangles around a hub (node 0): the hub's row has m + 1 entries, a rim node's four."""
    a = 2.0 * np.pi * np.arange(m) / m
    rim = np.stack([np.cos(a), np.sin(a)], axis=1) * (1.0 + 0.1 * np.sin(3 * a))[:, None]
    xy = np.concatenate([np.zeros((1, 2)), rim])
    k = np.arange(m)
    nodes = np.stack([np.zeros(m, dtype=np.int64), 1 + k, 1 + (k + 1) % m], axis=1).astype(np.int32)
    mesh = wl.Mesh(2, m + 1, nodes, xy[nodes], 4, 1.0)
    return wl.p2_mesh(mesh) if degree == 2 else mesh


@pytest.fixture(scope="module")
def pfc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06852_amd import pfc as lib
    return lib


# the hub's row: 96 (the longest staged), 97, 201; P2: the hub meets 2 m + 1 + m (rim edges) nodes
@pytest.mark.parametrize("m,degree", [(63, 1), (95, 1), (96, 1), (200, 1), (31, 2), (32, 2), (70, 2)])
def test_element_sums_at_row_lengths(pfc, m, degree):
    mesh = wheel(m, degree)
    n = mesh.n
    M, K = assembly.mass_stiffness(mesh)
    rng = np.random.default_rng(m)
    psi = -0.3 + 0.3 * rng.uniform(-1, 1, n)
    create = pfc.pfc_mesh_create_p2 if degree == 2 else pfc.pfc_mesh_create_p1
    h = create(2, n, mesh.elem_nodes, mesh.elem_coords)
    inst = pfc.pfc_instance_create(h, pfc.pfc_opts_default())
    try:
        # sums of at most 200 terms of one sign, each with a relative error of a few units in the last place
        rp, ci, mv, kv = pfc.pfc_mesh_export_csr(h)
        assert np.array_equal(rp, M.indptr) and np.array_equal(ci, M.indices)
        assert np.abs(mv - M.data).max() <= 1e-13 * np.abs(M.data).max()
        assert np.abs(kv - K.data).max() <= 1e-12 * np.abs(K.data).max()
        Nref = assembly.N_matrix(mesh, psi)
        Nd, g = dev(np.zeros(M.nnz)), dev(np.zeros(n))
        pfc.pfc_assemble_N(h, dev(psi), Nd)
        assert np.array_equal(Nref.indices, M.indices)
        assert np.abs(host(Nd) - Nref.data).max() <= 1e-13 * np.abs(Nref.data).max()
        pfc.pfc_load_psi3(h, dev(psi), g)
        assert blockerr(host(g), assembly.load_psi3(mesh, psi), 1) <= 1e-13
        r, tau, m11 = -0.35, 0.6, 1.0 / opfc.ROS3PW_GAMMA
        y, out = rng.normal(size=3 * n), dev(np.zeros(3 * n))
        pfc.pfc_apply_AR(inst, n, dev(psi), r, tau, m11, dev(y), out)
        assert blockerr(host(out), opfc.apply_AR(M, K, Nref, r, tau, m11, y)) <= 1e-12
        xk = np.concatenate([rng.normal(size=n), psi, rng.normal(size=n)])
        ys = 0.1 * rng.normal(size=(3, 3 * n))
        xi = xk + opfc.ROS3PW_A[(2, 1)] * ys[0]
        pfc.pfc_stage_rhs(inst, n, dev(xk), dev(ys.ravel()), 2, r, tau, out)
        b = opfc.stage_rhs_R(mesh, M, K, r, tau, xi, [ys[0][n:2 * n]], [opfc.ROS3PW_C[(2, 1)]])
        assert blockerr(host(out), b) <= 1e-12
    finally:
        pfc.pfc_instance_destroy(inst)
        pfc.pfc_mesh_destroy(h)


@pytest.mark.parametrize("m", [95, 130])
def test_step_on_long_rows(pfc, m):
    """A Rosenbrock step forms N and the loads inside the solver launches (8 entries a round)."""
    mesh = wheel(m)
    n = mesh.n
    M, K = assembly.mass_stiffness(mesh)
    r, tau = -0.35, 0.05
    psi = -0.3 + 0.05 * np.random.default_rng(m).uniform(-1, 1, n)
    x0 = opfc.consistent_init(mesh, M, K, r, psi)
    ref, _ = osolve.rosenbrock_run(mesh, M, K, x0, r, tau, 1, tol=1e-12)
    h = pfc.pfc_mesh_create_p1(2, n, mesh.elem_nodes, mesh.elem_coords)
    inst = pfc.pfc_instance_create(h, pfc.pfc_opts_default(outer_tol=1e-12))
    try:
        x = dev(x0)
        st, _ = pfc.pfc_rosenbrock_run(inst, n, x, r, -0.3, tau, 1, pfc.PFC_INIT_GIVEN)
        assert st == pfc.PFC_OK
        # both stop at a relative residual of 1e-12; the error of a solve is that times its condition
        assert np.linalg.norm(host(x) - ref) <= 1e-8 * np.linalg.norm(ref)
    finally:
        pfc.pfc_instance_destroy(inst)
        pfc.pfc_mesh_destroy(h)
