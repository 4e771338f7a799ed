"""A shape tuned on one batch meets a later batch of the same sizes on the same context, for which
its body is not valid: couplings beyond a byte, mixed class counts, a class larger than the tuned
workgroup.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_held import _layers

pytestmark = pytest.mark.gpu


def _lopsided(big, small, d, seed):
    """Two classes of `big` and `small` variables: the first `small` of each joined, d records each."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(small), d)
    j = (i + np.tile(np.arange(d), small)) % small
    w = rng.integers(1, 7, len(i)) * rng.choice([-1, 1], len(i))
    n = big + small
    return si.from_edges(n, i, big + j, w, rng.integers(-4, 5, n), np.arange(n) >= big, 2, 0)


PAIRS = {
    "beyond_bytes": (lambda: [_layers([40, 40], 6, 6, 1, 5), _layers([30, 30], 6, 6, 2, 5)],
                     lambda: [_layers([40, 40], 6, 70, 3, 5), _layers([30, 30], 6, 70, 4, 5)], 400),
    "mixed_class_counts": (lambda: [_layers([40, 40], 4, 6, 1, 4), _layers([30, 30], 4, 6, 2, 4)],
                           lambda: [_layers([40, 40], 4, 6, 3, 4), _layers([20, 20, 20], 2, 6, 4, 4)], 400),
    "three_classes": (lambda: [_layers([30, 30], 4, 6, 1, 4), _layers([30, 30], 4, 6, 2, 4)],
                      lambda: [_layers([20, 20, 20], 2, 6, 3, 4), _layers([20, 20, 20], 2, 6, 4, 4)], 400),
    "larger_class": (lambda: [_layers([400, 400], 3, 6, 1, 4)], lambda: [_lopsided(700, 100, 3, 2)], 60),
}


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("name", list(PAIRS))
def test_tuned_shape_meets_another_batch(name, graph):
    import paper_1706_07826_amd as spv
    first, second, reads = PAIRS[name]
    ctx = spv.Context(0)
    betas = si.linear_betas(0.05, 3.0, 12)
    for k, insts in enumerate((first(), second(), first())):
        x = max(oracle.x_max(i) for i in insts)
        assert (256 <= x <= 511) if (name == "beyond_bytes" and k == 1) else x <= 255
        n, seeds = [reads] * len(insts), [5 + b for b in range(len(insts))]
        print(f"[tuned] {name} batch {k} graph={graph} x_bound={x}", flush=True)
        sp, E = spv.spv_sample_batch(ctx, [spv.Problem.from_instance(i) for i in insts], betas, n, seeds,
                                     tune=k == 0, graph=graph)
        for b, inst in enumerate(insts):
            osp, oE = oracle.sa_sample(inst, betas, reads=reads, seed=seeds[b], threads=8)
            assert np.array_equal(sp[b].cpu().numpy(), osp) and np.array_equal(E[b].cpu().numpy(), oE), (k, b)
