"""Four large classes from global memory on both sides of the read count at which the held-sites body
gives way: the shape the launch reports, and the first and last reads against the oracle."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_held import _layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cls,reads,held", [(600, 3000, True), (600, 6000, False), (600, 6001, False),
                                            (800, 6000, True), (520, 6000, True)])
def test_four_classes(cls, reads, held):
    import paper_1706_07826_amd as spv
    inst = _layers([cls] * 4, 2, 3, 5, 2)
    betas = si.linear_betas(0.1, 2.0, 9)
    ctx = spv.Context(0)
    print(f"[held] four classes of {cls}, {reads} reads", flush=True)
    S, E = spv.spv_sample(ctx, spv.Problem.from_instance(inst), betas, reads, 7)
    assert (spv.spv_sample_last_shape(ctx)["global_instance"] == 0) == held
    S, E = S.cpu().numpy(), E.cpu().numpy()
    assert np.array_equal(E, oracle.energy(inst, S))
    for lo, hi in ((0, 12), (reads - 9, reads)):
        osp, oE = oracle.sa_sample(inst, betas, seed=7, r_begin=lo, r_end=hi)
        assert np.array_equal(S[lo:hi], osp) and np.array_equal(E[lo:hi], oE)
