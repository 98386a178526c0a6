"""pfc_instance_launch_stats counts the launches that advanced the instance, on the device: the number follows
from the iteration counts alone, not from the launches a graph holds or from when the host sees the end
(needs a GPU)."""
import numpy as np
import pytest

from helpers import Problem, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pfc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06852_amd import pfc as lib
    return lib


# a grid without the two-iteration form's blocks (ranges of grid lines, float64), and one of blocks
@pytest.mark.parametrize("N,prec", [(33, 0), (64, 0), (64, 1)])
@pytest.mark.parametrize("spl", [1, 2])
@pytest.mark.parametrize("ticks", [2, 64, 128])
def test_launches_follow_from_the_iterations(pfc, N, prec, spl, ticks):
    P = Problem(2, N, 0.2, seed=51)
    inst = pfc.pfc_instance_create(P.gpu_mesh(), pfc.pfc_opts_default(precision=prec, pcg_steps_per_launch=spl,
                                                                      ticks_per_graph=ticks))
    try:
        v = dev(np.random.default_rng(51).normal(size=3 * P.n))
        z = dev(np.zeros(3 * P.n))
        for counts in ([8, 10, 20, 25, 8], [3, 1, 4, 5, 2]):
            pfc.pfc_apply_pch(inst, P.n, 0.4, v, z, fixed_counts=counts)
            launches, graphs = pfc.pfc_instance_launch_stats(inst)
            # a solve: its set-up and first product, and a launch an iteration; two iterations a launch: the
            # set-up, a launch a pair, where the last pair of the first four is one launch with the next
            # set-up in the block form; then the launch that stores the result and the one that ends
            if spl == 1:
                want = sum(2 + c for c in counts) + 2
            else:
                want = sum(1 + (c + 1) // 2 for c in counts) + 2 - (4 if N % 64 == 0 else 0)
            assert launches == want, (counts, launches, want)
            assert want <= graphs * ticks
    finally:
        pfc.pfc_instance_destroy(inst)
        P.close()
