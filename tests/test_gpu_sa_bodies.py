"""GPU parity of the byte-parallel bodies that read their records from LDS (one and two words per
lane, 4, 6, 8 and any number of records a site), in one launch and streamed, with the held-sites body
that otherwise takes such problems switched off; the launch's own report names the body."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_held import _layers

pytestmark = pytest.mark.gpu

INSTANCES = {"two": lambda: _layers([40, 40], 2, 6, 1, 5), "four": lambda: _layers([40, 37], 4, 6, 2, 0),
             "six": lambda: si.chimera(3, seed=4), "eight": lambda: _layers([33, 33], 8, 6, 3, 5),
             "four_classes": lambda: _layers([30] * 4, 2, 6, 4, 5)}


@pytest.mark.parametrize("stream", [0, 8])
@pytest.mark.parametrize("words", [1, 2])
@pytest.mark.parametrize("name", list(INSTANCES))
def test_bodies(monkeypatch, name, words, stream):
    import paper_1706_07826_amd as spv
    inst = INSTANCES[name]()
    assert oracle.x_max(inst) <= 255
    env = dict(SPVAR_SA_HELD=0, SPVAR_SA_WPL=words, SPVAR_SA_THREADS=256, SPVAR_SA_STREAM=stream)
    for k, v in env.items():
        monkeypatch.setenv(k, str(v))
    ctx = spv.Context(0)
    betas = np.concatenate([[0.0], si.linear_betas(0.05, 3.0, 47)])
    print(f"[bodies] {name} words={words} stream={stream}", flush=True)
    S, E = spv.spv_sample(ctx, spv.Problem.from_instance(inst), betas, 150, 23)
    shape = spv.spv_sample_last_shape(ctx)
    assert shape["words_per_lane"] == words and (shape["chunks"] > 1) == (stream > 0)
    assert shape["threads"] == 256 and not shape["global_instance"]
    osp, oE = oracle.sa_sample(inst, betas, reads=150, seed=23, threads=8)
    assert np.array_equal(S.cpu().numpy(), osp) and np.array_equal(E.cpu().numpy(), oE)
