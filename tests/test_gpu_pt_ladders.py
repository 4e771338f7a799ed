"""GPU parity of tempering on ladders that are no multiple of four, split over workgroups or in one
(each chain's quads then start at another slot), and of one-group runs beyond the device's resident
workgroups, bit for bit against the CPU oracle; resumed too."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spv():
    import paper_1706_07826_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(spv):
    return spv.Context(0)


def _check(got, want):
    for key in ("final_spins", "final_E", "top_E", "top_count", "top_spins"):
        assert np.array_equal(got[key].cpu().numpy(), want[key]), key


GAUSS = lambda s: si.cubic_lattice(4, "gauss", seed=s, scale_log2=10)
CASES = [
    # name, instance, K, runs, chains, sweeps, icm, groups (0: the planner's), big
    ("K5_two_groups", lambda: GAUSS(1), 5, 3, 1, 60, None, 2, 0),
    ("K5_planned", lambda: GAUSS(2), 5, 3, 1, 60, None, 0, 0),
    ("K6_single_slots", lambda: GAUSS(3), 6, 3, 2, 60, (0, 6), 6, 0),
    ("K6_single_slots_packed", lambda: GAUSS(4), 6, 3, 2, 60, (0, 6), 6, 1),
    ("K7_single_slots_packed_window", lambda: GAUSS(5), 7, 3, 2, 61, (2, 6), 7, 1),
    ("K7_half_quads", lambda: GAUSS(6), 7, 3, 2, 61, (0, 7), 4, 0),
    ("K7_half_quads_big", lambda: GAUSS(7), 7, 2, 2, 61, (1, 7), 4, 1),
    ("K13_three_chains", lambda: si.cubic_lattice(4, "pm1", seed=8), 13, 3, 3, 50, None, 2, 0),
    ("K14_two_groups_icm", lambda: GAUSS(9), 14, 2, 2, 50, (0, 14), 2, 0),
    ("K14_two_groups_icm_big", lambda: GAUSS(10), 14, 2, 2, 50, (3, 12), 2, 1),
    ("K9_sparse_any_degree", lambda: si.random_sparse(41, 3.0, seed=11), 9, 3, 2, 50, (0, 9), 9, 0),
    ("K9_sparse_any_degree_big", lambda: si.random_sparse(41, 3.0, seed=12), 9, 3, 2, 50, (0, 9), 9, 1),
    ("K10_three_digits", lambda: si.random_sparse(30, 9.0, seed=13, scale_log2=14,
                                                  dist=("uniform_nonzero", 32767)), 10, 2, 2, 40, (0, 10), 5, 0),
    ("K26_planned_icm", lambda: si.cubic_lattice(6, "gauss", seed=14, scale_log2=10), 26, 3, 2, 40, (0, 26), 0, 0),
    ("K26_planned", lambda: si.cubic_lattice(6, "gauss", seed=15, scale_log2=10), 26, 3, 2, 40, None, 0, 0),
    ("K2_icm", lambda: GAUSS(16), 2, 3, 2, 40, (0, 2), 0, 0),
    ("K1", lambda: GAUSS(17), 1, 3, 2, 20, (0, 1), 0, 0),
]


@pytest.mark.parametrize("name,make,K,runs,chains,sweeps,icm,groups,big", CASES, ids=[c[0] for c in CASES])
def test_ladders(spv, ctx, monkeypatch, name, make, K, runs, chains, sweeps, icm, groups, big):
    inst = make()
    print(f"[ladders] {name} K={K} runs={runs} chains={chains} G={groups} big={big}", flush=True)
    monkeypatch.setenv("SPVAR_PT_GROUPS", str(groups))
    monkeypatch.setenv("SPVAR_PT_BIG", str(big))
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0 if inst.scale_log2 else 3.0, K)
    got = spv.spv_pt_sample(ctx, P, betas, runs, chains, sweeps, seed=90 + K, icm=icm)
    want = oracle.pt_sample(inst, betas, runs, chains, sweeps, seed=90 + K, icm=icm, threads=8)
    _check(got, want)
    more = 15
    got = spv.spv_pt_sample(ctx, P, betas, runs, chains, more, seed=90 + K, sweep_offset=sweeps, icm=icm, resume=got)
    want = oracle.pt_sample(inst, betas, runs, chains, more, seed=90 + K, sweep_offset=sweeps, icm=icm, resume=want,
                            threads=8)
    _check(got, want)


@pytest.mark.parametrize("K,chains,icm", [(8, 1, None), (5, 2, None), (8, 2, (0, 8)), (5, 2, (1, 4))])
def test_many_runs(spv, ctx, K, chains, icm):
    """More runs than workgroups stay resident: one group a run, none waits for another."""
    inst = GAUSS(18)
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0, K)
    print(f"[ladders] 2100 runs K={K} chains={chains} icm={icm}", flush=True)
    got = spv.spv_pt_sample(ctx, P, betas, 2100, chains, 12, seed=7, icm=icm)
    want = oracle.pt_sample(inst, betas, 2100, chains, 12, seed=7, icm=icm, threads=8)
    _check(got, want)
