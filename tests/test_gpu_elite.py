"""Elite selection where the rows held per lane change (1024, 4096, 16384 rows, then none held), over
ties, equal keys and keys of every byte, and the gauge's table cleared by few and by many workgroups:
bit for bit against the oracle."""
import numpy as np
import pytest

import spvar_inputs as si
from .test_gpu_persist import _compare, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

KEYS = {
    "ties": lambda rng, R: rng.integers(-3, 3, R),
    "equal": lambda rng, R: np.full(R, 7),
    "two_bytes": lambda rng, R: rng.integers(-20000, 20000, R),
    "full": lambda rng, R: rng.integers(-2 ** 62, 2 ** 62, R),
}


@pytest.mark.parametrize("keys", list(KEYS))
@pytest.mark.parametrize("R", [63, 64, 1023, 1024, 1025, 4096, 4097, 16384, 16385, 33000])
def test_elite(spv, ctx, R, keys):  # noqa: F811
    inst = si.random_sparse(23, 3.0, seed=6)
    rng = np.random.default_rng(R)
    S = si.random_spins(R, inst.n, seed=R)
    E = KEYS[keys](rng, R).astype(np.int64)
    for eps, theta in ((0.05, 0.6), (1.0, 0.5), (1.5 / R, 1.0)):
        print(f"[elite] R={R} {keys} eps={eps}", flush=True)
        _compare(spv, ctx, inst, S, E, eps, theta, 0)


@pytest.mark.parametrize("n,R", [(2, 5000), (5, 3), (64, 70), (65, 4000), (700, 1), (700, 2000)])
def test_gauge_table(spv, ctx, n, R):  # noqa: F811
    inst = si.random_sparse(n, 1.0, seed=n)
    S = si.random_spins(R, inst.n, seed=R)
    S[:, 1::3] = S[:, :1]  # a class of equal columns
    E = np.random.default_rng(n).integers(-50, 50, R)
    for again in range(2):
        print(f"[gauge] n={n} R={R} {again}", flush=True)
        _compare(spv, ctx, inst, S, E, 0.7, 0.9, 1)
