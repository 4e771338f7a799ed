"""Cluster moves of the one-workgroup tempering kernel, bit for bit against the CPU oracle: found by
growth, by the union-find, and by a growth that is given up for the union-find, over sizes around both
lines (128 and 256 sites), few and many small components, and more than 64 slots a wavefront."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_ladders import _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _cliques(count, size, seed):
    rng = np.random.default_rng(seed)
    a, b = np.triu_indices(size, 1)
    ei = np.concatenate([a * count + c for c in range(count)])
    ej = np.concatenate([b * count + c for c in range(count)])
    w = rng.integers(1, 7, len(ei)) * rng.choice([-1, 1], len(ei))
    n = count * size
    return si.from_edges(n, ei, ej, w, rng.integers(-2, 3, n), np.repeat(np.arange(size), count), size, 0)


def _path(n, seed):
    rng = np.random.default_rng(seed)
    i = np.arange(n - 1)
    return si.from_edges(n, i, i + 1, rng.choice([-2, -1, 1, 2], n - 1), rng.integers(-1, 2, n), np.arange(n) % 2, 2, 0)


CASES = {
    "cliques": (lambda: _cliques(50, 5, 1), 6, 3, None),
    "cliques_few_sites": (lambda: _cliques(25, 5, 2), 6, 3, None),
    # small and large components beside each other: growths given up
    "cube_and_cliques": (lambda: si.disjoint_union([si.cubic_lattice(5, "pm1", seed=3), _cliques(20, 5, 4)]), 8, 3, None),
    "cube6": (lambda: si.cubic_lattice(6, "gauss", seed=5, scale_log2=10), 5, 2, (1, 5)),
    "cube7": (lambda: si.cubic_lattice(7, "gauss", seed=6, scale_log2=10), 6, 2, None),
    "sites256": (lambda: _path(256, 7), 5, 2, None),
    "sites257": (lambda: _path(257, 8), 5, 2, None),
    "sites129": (lambda: _path(129, 9), 5, 2, None),
    "random600": (lambda: si.random_sparse(600, 3.0, seed=10), 3, 2, None),
    "many_slots": (lambda: _path(140, 11), 290, 1, None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_clusters(spv, ctx, monkeypatch, name):  # noqa: F811
    make, K, runs, icm = CASES[name]
    inst = make()
    monkeypatch.setenv("SPVAR_PT_SPLIT", "0")
    print(f"[clusters] {name} n={inst.n} K={K}", flush=True)
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.1, 5.0 if inst.scale_log2 else 2.0, K)
    sweeps = 25 if K > 64 else 120
    got = spv.spv_pt_sample(ctx, P, betas, runs, 2, sweeps, seed=8, icm=icm or (0, K))
    want = oracle.pt_sample(inst, betas, runs, 2, sweeps, seed=8, icm=icm or (0, K), threads=8)
    _check(got, want)
