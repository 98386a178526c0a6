"""The operator applies where the result replaces the vector that holds psi_k: the same A^R y as with psi_k
in memory of its own (needs a GPU)."""
import numpy as np
import pytest

from helpers import Problem, blockerr, dev, host
from oracle import assembly, pfc as opfc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pfc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06852_amd import pfc as lib
    return lib


# many workgroups (2D 96^2: 144 slices), 3D, P2
@pytest.mark.parametrize("dim,N,degree", [(2, 96, 1), (3, 9, 1), (2, 12, 2)])
@pytest.mark.parametrize("at", [0.0, 1.0, 2.5])  # where psi_k begins in out, in units of n; 2.5: half beyond its end
def test_out_overlaps_psi(pfc, dim, N, degree, at):
    import torch
    P = Problem(dim, N, 0.1, amp=0.2, seed=61, degree=degree)
    n = P.n
    y = np.random.default_rng(61).normal(size=3 * n)
    r, tau, m11 = -0.35, 0.7, 1.0 / opfc.ROS3PW_GAMMA
    ref = opfc.apply_AR(P.M, P.K, assembly.N_matrix(P.mesh, P.psi), r, tau, m11, y)
    inst = pfc.pfc_instance_create(P.gpu_mesh(), pfc.pfc_opts_default())
    o = int(at * n)

    def buffers():
        buf = dev(np.zeros(4 * n))
        buf[o:o + n] = dev(P.psi)
        return buf[o:o + n], buf[:3 * n]

    try:
        psi, out = buffers()
        pfc.pfc_apply_AR(inst, n, psi, r, tau, m11, dev(y), out)
        assert blockerr(host(out), ref) <= 1e-12
        psi, out = buffers()
        pfc.pfc_apply_AR_noalloc(P.gpu_mesh(), n, psi, r, tau, m11, dev(y), out)
        torch.cuda.synchronize()
        assert blockerr(host(out), ref) <= 1e-12
        x = dev(np.concatenate([y[:n], P.psi, y[:n]]))
        pfc.pfc_apply_AR_x(inst, n, x, r, tau, m11, dev(y), x)
        assert blockerr(host(x), ref) <= 1e-12
    finally:
        pfc.pfc_instance_destroy(inst)
        P.close()
