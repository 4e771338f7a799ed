"""Serving under a budget that holds a tempering request as one workgroup a run, but not its split
ladder: requests off the multiples of four, and ones of one group a run, are still accepted and exact;
a multiple of four whose split does not fit is still refused."""
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_ladders import GAUSS, _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _lds(spv, ctx, P, betas, runs, chains, icm):  # noqa: F811
    srv = spv.Server(ctx, slots=1)
    res, keep = srv.wait(srv.submit_pt(P, betas, runs, chains, 3, 5, icm=icm))
    srv.close()
    return res.lds_bytes


# (name, K, runs, chains, icm)
CASES = [("off_icm", 26, 2, 2, (0, 26)), ("off", 30, 1, 2, None), ("one_group", 8, 200, 1, None)]


@pytest.mark.parametrize("name,K,runs,chains,icm", CASES, ids=[c[0] for c in CASES])
def test_budget_of_one_workgroup(spv, ctx, monkeypatch, name, K, runs, chains, icm):  # noqa: F811
    inst = GAUSS(31)
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0, K)
    print(f"[serving] {name}", flush=True)
    split = _lds(spv, ctx, P, betas, runs, chains, icm)
    monkeypatch.setenv("SPVAR_PT_SPLIT", "0")
    single = _lds(spv, ctx, P, betas, runs, chains, icm)
    monkeypatch.delenv("SPVAR_PT_SPLIT")
    assert single < split
    srv = spv.Server(ctx, slots=2, lds_budget=single)
    got = [srv.wait(srv.submit_pt(P, betas, runs, chains, 30, seed, icm=icm)) for seed in (7, 8)]
    with pytest.raises(spv.SpvError, match="EBUDGET"):
        srv.submit_pt(P, betas, 2 * runs, chains, 30, 7, icm=icm)
    srv.close()
    for seed, (res, keep) in zip((7, 8), got):
        assert res.lds_bytes == single
        _check(keep, oracle.pt_sample(inst, betas, runs, chains, 30, seed=seed, icm=icm, threads=8))


def test_split_multiple_of_four_is_refused(spv, ctx):  # noqa: F811
    P = spv.Problem.from_instance(GAUSS(32))
    betas = si.geometric_betas(0.2, 5.0, 16)
    srv = spv.Server(ctx, slots=1, lds_budget=_lds(spv, ctx, P, betas, 2, 2, (0, 16)) - 1)
    with pytest.raises(spv.SpvError, match="EBUDGET"):
        srv.submit_pt(P, betas, 2, 2, 30, 7, icm=(0, 16))
    srv.close()


@pytest.mark.parametrize("L,K,chains,split", [(4, 10, 1, False), (4, 14, 2, True), (5, 10, 2, False), (6, 10, 2, True),
                                              (4, 30, 1, True), (7, 10, 1, False)])
def test_which_ladders_are_split(spv, ctx, monkeypatch, L, K, chains, split):  # noqa: F811
    """Ladders off the multiples of four, without cluster moves: in one group with at most three
    quads and few words a sweep, else split (the footprint counts every group's copy)."""
    P = spv.Problem.from_instance(si.cubic_lattice(L, "gauss", seed=3, scale_log2=10))
    betas = si.geometric_betas(0.2, 5.0, K)
    planned = _lds(spv, ctx, P, betas, 2, chains, None)
    monkeypatch.setenv("SPVAR_PT_GROUPS", "1")
    one = _lds(spv, ctx, P, betas, 2, chains, None)
    assert (planned > one) == split
