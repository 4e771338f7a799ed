"""Tempering launches on both sides of the rules that choose between the one-workgroup kernel, one
group of the split kernel (with narrower workgroups where more runs are then resident) and a split
ladder, bit for bit against the CPU oracle."""
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_clusters import _path
from .test_gpu_pt_ladders import GAUSS, _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CUBE6 = lambda: si.cubic_lattice(6, "gauss", seed=3, scale_log2=10)
CASES = [
    # name, instance, K, runs, chains, sweeps, icm
    ("few_sites_off_one_workgroup", lambda: _path(40, 1), 13, 5, 2, 30, None),
    ("few_sites_off_split", lambda: _path(50, 2), 30, 5, 2, 30, None),
    ("short_off_one_workgroup", lambda: _path(110, 3), 6, 5, 2, 30, None),
    ("short_off_one_group", lambda: _path(300, 4), 6, 5, 2, 30, None),
    ("few_sites_one_workgroup", lambda: _path(40, 5), 8, 300, 2, 12, None),
    ("short_one_workgroup", lambda: _path(120, 11), 8, 5, 1, 30, None),
    ("short_split", lambda: _path(130, 12), 8, 5, 1, 30, None),
    ("narrower_workgroups", lambda: _path(250, 6), 16, 600, 2, 6, None),
    ("narrower_workgroups_off", CUBE6, 6, 700, 2, 6, None),
    ("fewer_rounds_in_one_workgroup", lambda: si.cubic_lattice(3, "gauss", seed=7, scale_log2=10), 32, 300, 2, 12, None),
    ("two_rounds_either_way", CUBE6, 32, 600, 1, 6, None),
    ("three_groups_for_two", lambda: _path(120, 8), 10, 100, 2, 20, (0, 10)),
    ("few_sites_icm", lambda: _path(40, 9), 10, 100, 2, 20, (0, 10)),
    ("two_slots_icm", lambda: _path(120, 10), 2, 20, 2, 20, (0, 2)),
]


@pytest.mark.parametrize("name,make,K,runs,chains,sweeps,icm", CASES, ids=[c[0] for c in CASES])
def test_routes(spv, ctx, name, make, K, runs, chains, sweeps, icm):  # noqa: F811
    inst = make()
    print(f"[routes] {name} n={inst.n} K={K} runs={runs}", flush=True)
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 4.0 if inst.scale_log2 else 2.0, K)
    got = spv.spv_pt_sample(ctx, P, betas, runs, chains, sweeps, seed=12, icm=icm)
    want = oracle.pt_sample(inst, betas, runs, chains, sweeps, seed=12, icm=icm, threads=8)
    _check(got, want)
