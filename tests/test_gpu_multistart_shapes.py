"""The batched solving sample of a multi-start call takes the narrow shape (a workgroup just wide
enough for one colour class x 2 quad words) exactly where the held-sites body does not serve the
residual problems; results against the oracle."""
import numpy as np
import pytest

import spvar_inputs as si
from .test_gpu_held import _layers
from .test_gpu_multistart import _run, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _ring(n, seed):
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    return si.from_edges(n, i, (i + 1) % n, rng.integers(1, 7, n) * rng.choice([-1, 1], n), rng.integers(-3, 4, n),
                         i % 2, 2, 0)


CASES = {
    "held": (lambda: si.chimera(3, seed=2), True),
    "two_digits": (lambda: si.cubic_lattice(4, "gauss", seed=3, scale_log2=10), False),
    "beyond_bytes": (lambda: _layers([40, 40], 6, 70, 3, 5), False),
    "five_classes": (lambda: _layers([12] * 5, 1, 6, 4, 3), False),
    "two_records": (lambda: _ring(60, 5), False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_shape(spv, ctx, name):  # noqa: F811
    make, held = CASES[name]
    inst = make()
    print(f"[shapes] {name} n={inst.n}", flush=True)
    got = _run(spv, ctx, inst, si.linear_betas(0.05, 1.0, 12), seed=3, starts=3, fixing_reads=60,
               solving_reads=41, elite_frac=0.5, threshold=1.0)
    n_left = got["info"][:, 3]
    assert (n_left > 0).all()
    shape = spv.spv_batch_last_shape(ctx)
    if held:
        assert shape["quads_per_item"] == 0
    else:
        cls = int(max((n_left + inst.n_colours - 1) // inst.n_colours))
        assert (shape["threads"], shape["quads_per_item"]) == (min(256, (2 * cls + 63) // 64 * 64), 2)
