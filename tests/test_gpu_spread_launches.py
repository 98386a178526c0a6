"""Launches that serve one instance on more workgroups than its team (meshes of at most 2048 slices of 64
rows) leave a partial sum per slice, added up in the team's order: the bits of the same instance in a batch,
whose launches keep the teams (needs a GPU)."""
import numpy as np
import pytest

import workloads as wl
from helpers import Problem, dev, host, rel
from oracle import pfc as opfc, solve as osolve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pfc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06852_amd import pfc as lib
    return lib


# one slice and two (the second of 17 rows); 16 and 18 slices (a full workgroup; teams of 9 slices a
# workgroup); rows of 15 entries, by columns from the grid or from memory; P2 (slices dealt round robin);
# 257 slices (two a workgroup); 2048 (the most) and 2059 (the team again)
CASES = [(2, 8, 0.2, 1, 0, 1), (2, 9, 0.0, 1, 1, 1), (2, 32, 0.2, 1, 1, 1), (2, 33, 0.0, 1, 0, 1), (3, 13, 0.2, 1, 0, 1),
         (3, 13, 0.0, 1, 1, 1), (2, 33, 0.2, 1, 0, 0), (2, 10, 0.0, 2, 0, 1), (2, 17, 0.2, 2, 1, 1), (2, 128, 0.0, 1, 0, 1),
         (2, 362, 0.0, 1, 1, 1), (2, 363, 0.0, 1, 0, 1)]


@pytest.mark.parametrize("dim,N,jit,degree,prec,grid", CASES)
def test_spread_launches_equal_team_launches(pfc, dim, N, jit, degree, prec, grid):
    _alone_equals_batch(pfc, Problem(dim, N, jit, seed=41, degree=degree), precision=prec, grid_columns=grid)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("opts", [dict(model=1), dict(schur_variant=1), dict(single_reduction=0), dict(shared_ops=1)],
                         ids=lambda o: next(iter(o)))
def test_spread_launches_options(pfc, opts, prec):
    _alone_equals_batch(pfc, Problem(2, 33, 0.2, seed=44), precision=prec, **opts)


def _alone_equals_batch(pfc, P, **opts):
    Q = Problem(2, 10, 0.0, seed=42)
    prm = wl.draw_params(2, 700)
    insts, states = [], []
    try:
        for p, X in zip(prm, (P, Q)):
            o = pfc.pfc_opts_default(rows_per_thread=1, pcg_steps_per_launch=1, **opts)
            insts.append(pfc.pfc_instance_create(X.gpu_mesh(), o))
            states.append(np.concatenate([np.zeros(X.n), wl.psi0(X.n, p.psibar, 0.01, seed=p.seed), np.zeros(X.n)]))
        alone = []
        for inst, p, X, s in zip(insts, prm, (P, Q), states):
            a = dev(s)
            st, _ = pfc.pfc_rosenbrock_run(inst, X.n, a, p.r, p.psibar, p.tau, 1)
            assert st == pfc.PFC_OK
            alone.append(host(a))
        batch = [dev(s) for s in states]
        st, _ = pfc.pfc_batch_run(insts, [P.n, Q.n], batch, [p.r for p in prm], [p.psibar for p in prm],
                                  [p.tau for p in prm], 1)
        assert st >= 0
        for k in range(2):
            assert np.array_equal(host(batch[k]), alone[k]), k
    finally:
        for i in insts:
            pfc.pfc_instance_destroy(i)
        P.close()
        Q.close()


@pytest.mark.parametrize("N", [9, 33, 100])
def test_spread_row_ranges_against_oracle(pfc, N):
    """Two iterations per launch on ranges of grid lines of one slice each (float64): the oracle's stage
    solve to the accuracy of two solves at relative residual 1e-8."""
    P = Problem(2, N, 0.2, seed=43)
    p = wl.draw_params(1, 800)[0]
    inst = pfc.pfc_instance_create(P.gpu_mesh(), pfc.pfc_opts_default(precision=0))
    try:
        assert pfc.pfc_instance_config(inst)["pcg_steps_per_launch"] == 2
        psi = wl.psi0(P.n, p.psibar, 0.01, seed=p.seed)
        s = dev(np.concatenate([np.zeros(P.n), psi, np.zeros(P.n)]))
        st, _ = pfc.pfc_rosenbrock_run(inst, P.n, s, p.r, p.psibar, p.tau, 1)
        assert st == pfc.PFC_OK
        x0 = opfc.consistent_init(P.mesh, P.M, P.K, p.r, psi)
        xr, _ = osolve.rosenbrock_run(P.mesh, P.M, P.K, x0, p.r, p.tau, 1, tol=1e-8)
        assert rel(host(s), xr) <= 1e-6
    finally:
        pfc.pfc_instance_destroy(inst)
        P.close()
