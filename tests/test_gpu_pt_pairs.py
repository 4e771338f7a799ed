"""Replica exchange of more slot pairs than a narrow workgroup has threads (256), on a handful of
sites, in the one-workgroup kernel and in the split one, bit for bit against the CPU oracle."""
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_ladders import _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [
    # name, sites, K, chains, icm, environment
    ("one_workgroup_320", 2, 10, 64, None, {"SPVAR_PT_SPLIT": 0}),
    ("one_workgroup_300_icm", 5, 300, 2, (0, 300), {"SPVAR_PT_SPLIT": 0}),
    ("one_group_320", 2, 10, 64, None, {}),
    ("one_group_300", 5, 200, 3, None, {}),
    ("one_group_384", 2, 12, 64, None, {"SPVAR_PT_GROUPS": 1}),
    ("two_groups_384", 3, 16, 64, None, {"SPVAR_PT_GROUPS": 2}),
]


@pytest.mark.parametrize("name,n,K,chains,icm,env", CASES, ids=[c[0] for c in CASES])
def test_pairs(spv, ctx, monkeypatch, name, n, K, chains, icm, env):  # noqa: F811
    inst = si.from_edges(n, range(n - 1), range(1, n), [3, -2, 1, 2][:n - 1], [1, 0, -1, 2, 0][:n],
                         [i % 2 for i in range(n)], 2, 0)
    for k, v in env.items():
        monkeypatch.setenv(k, str(v))
    print(f"[pairs] {name} n={n} K={K} chains={chains}", flush=True)
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.05, 1.5, K)
    got = spv.spv_pt_sample(ctx, P, betas, 2, chains, 25, seed=3, icm=icm)
    want = oracle.pt_sample(inst, betas, 2, chains, 25, seed=3, icm=icm, threads=8)
    _check(got, want)
