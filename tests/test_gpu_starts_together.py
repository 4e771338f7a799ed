"""The starts of a multi-start call reduced and recombined in the same launches: all together, in
groups of a few and one by one, with starts of different sizes, empty ones, and more components than
the partial energies keep in LDS (8192)."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_multistart import _run, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _singles(n, seed):
    """Biased variables without couplers but one."""
    rng = np.random.default_rng(seed)
    return si.from_edges(n, [0], [1], [1], rng.integers(-1, 2, n), np.arange(n) % 2, 2, 0)


CASES = {
    "union": (lambda: si.disjoint_union([si.chimera(1, seed=2), si.random_sparse(25, 2.0, seed=3),
                                         si.random_sparse(12, 1.5, seed=4)], perm_seed=2),
              dict(starts=7, fixing_reads=50, solving_reads=41, elite_frac=0.1, threshold=0.9, merge=True), 40),
    "corr": (lambda: si.chimera(3, seed=33, h_zero=True),
             dict(starts=5, corr_reads=37, fixing_reads=29, solving_reads=23, elite_frac=0.2, threshold=1.0,
                  corr_elite_frac=0.2, merge=True), 40),
    "some_empty": (lambda: si.random_sparse(9, 2.0, seed=8),
                   dict(starts=12, fixing_reads=6, solving_reads=5, elite_frac=0.6, threshold=0.8, merge=True), 3),
    # (SQA: the batched SA launch has no room for so many variables)
    "many_components": (lambda: _singles(8600, 4),
                        dict(starts=3, fixing_reads=9, solving_reads=6, elite_frac=1.0, threshold=1.0, merge=True,
                             gammas=np.geomspace(3.0, 1.0, 2), trotter=8), 2),
}


@pytest.mark.parametrize("kb", [None, 0, 200])
@pytest.mark.parametrize("name", list(CASES))
def test_starts_together(spv, ctx, monkeypatch, name, kb):  # noqa: F811
    make, kw, sweeps = CASES[name]
    if kb is not None:
        monkeypatch.setenv("SPVAR_MS_TOGETHER_KB", str(kb))
    inst = make()
    betas = si.linear_betas(0.05, 0.1 if name == "many_components" else 3.0, sweeps)
    print(f"[together] {name} n={inst.n} kb={kb}", flush=True)
    got = _run(spv, ctx, inst, betas, seed=41, **kw)
    if name == "some_empty":
        assert (got["info"][:, 3] == 0).any() and (got["info"][:, 3] > 0).any()
    if name == "many_components":
        assert (got["info"][:, 5] > 8192).all()
