"""GPU parity of tempering over the words a group keeps per site (1, 2, 4, .. 32, and no power of two:
the energy sums and the in-group swaps work word by word), over states stored by words and by bytes,
and beyond the sizes whose energy sums fit 32 bits, bit for bit against the CPU oracle."""
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_ladders import _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CUBE = lambda L, s: si.cubic_lattice(L, "gauss", seed=s, scale_log2=10)
CASES = [
    # name, instance, K, runs, chains, sweeps, icm, groups
    ("one_word", lambda: CUBE(4, 1), 8, 2, 1, 60, None, 2),
    ("two_words", lambda: CUBE(4, 2), 16, 2, 1, 60, None, 2),
    ("three_words", lambda: CUBE(4, 3), 24, 2, 1, 60, None, 2),
    ("four_words_odd_cube", lambda: CUBE(5, 4), 32, 2, 1, 60, None, 2),
    ("eight_words", lambda: CUBE(4, 5), 32, 2, 1, 60, None, 1),
    ("sixteen_words_two_chains", lambda: CUBE(4, 6), 32, 2, 2, 40, None, 1),
    ("thirty_two_words_two_chains", lambda: CUBE(4, 7), 64, 1, 2, 40, None, 1),
    ("two_words_two_chains_icm", lambda: CUBE(6, 8), 16, 2, 2, 40, (0, 16), 4),
    ("four_pairs_odd_cube_icm", lambda: CUBE(5, 9), 16, 2, 2, 40, (2, 14), 4),
    ("pm1_cube", lambda: si.cubic_lattice(6, "pm1", seed=10), 16, 3, 1, 60, None, 2),
    ("sums_in_64_bits", lambda: CUBE(21, 11), 8, 1, 1, 4, None, 2),
    ("sums_in_64_bits_packed", lambda: CUBE(21, 12), 4, 1, 2, 4, (0, 4), 4),
    ("three_digits", lambda: si.random_sparse(60, 9.0, seed=13, scale_log2=14, dist=("uniform_nonzero", 32767)),
     16, 2, 1, 40, None, 2),
]


@pytest.mark.parametrize("name,make,K,runs,chains,sweeps,icm,groups", CASES, ids=[c[0] for c in CASES])
def test_words(spv, ctx, monkeypatch, name, make, K, runs, chains, sweeps, icm, groups):  # noqa: F811
    inst = make()
    print(f"[words] {name} n={inst.n} K={K} G={groups}", flush=True)
    monkeypatch.setenv("SPVAR_PT_GROUPS", str(groups))
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0 if inst.scale_log2 else 3.0, K)
    got = spv.spv_pt_sample(ctx, P, betas, runs, chains, sweeps, seed=40 + K, icm=icm)
    want = oracle.pt_sample(inst, betas, runs, chains, sweeps, seed=40 + K, icm=icm, threads=8)
    _check(got, want)
