"""SQA parity over record counts with loops of their own (one to three, six) and around them, at the
smallest and a wide slice count, in LDS and in global memory, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_fields import _complete_bipartite

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 6, 7])
@pytest.mark.parametrize("j", [3, 900])
@pytest.mark.parametrize("P", [8, 40])
@pytest.mark.parametrize("big", ["0", "1"])
def test_records(monkeypatch, d, j, P, big):
    import paper_1706_07826_amd as spv
    monkeypatch.setenv("SPVAR_SQA_BIG", big)
    inst = _complete_bipartite(d, j, 0, 3 + d, 0 if j == 3 else 11)
    betas, gammas = si.linear_betas(0.2, 2.0, 12), np.geomspace(3.0, 0.05, 12)
    print(f"[sqa] d={d} j={j} P={P} big={big}", flush=True)
    sp, E = spv.spv_sqa_sample(spv.Context(0), spv.Problem.from_instance(inst), betas, gammas, P, 5, 9)
    osp, oE, _ = oracle.sqa_sample(inst, betas, gammas, P, reads=5, seed=9)
    assert np.array_equal(sp.cpu().numpy(), osp) and np.array_equal(E.cpu().numpy(), oE)
