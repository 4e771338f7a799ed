"""Split ladders that are no multiple of four never report an abandoned wait: with a spin limit of 0
(a workgroup gives up unless its neighbour has published already) every run still equals the CPU
oracle bit for bit, fresh, resumed and resumed in place; and so with another stream's work on the
device."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si
from .test_gpu_pt_ladders import GAUSS, _check, ctx, spv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [
    # name, K, runs, chains, icm, groups
    ("two_groups", 5, 3, 1, None, 2),
    ("half_quads_icm", 7, 3, 2, (0, 7), 4),
    ("single_slots_icm", 6, 5, 2, (0, 6), 6),
    ("planned", 26, 4, 2, None, 0),
    ("planned_icm", 26, 4, 2, (0, 26), 0),
]


@pytest.mark.parametrize("spin", [0, 1 << 24])
@pytest.mark.parametrize("name,K,runs,chains,icm,groups", CASES, ids=[c[0] for c in CASES])
def test_abandoned_waits(spv, ctx, monkeypatch, name, K, runs, chains, icm, groups, spin):  # noqa: F811
    inst = GAUSS(23)
    print(f"[redo] {name} spin={spin}", flush=True)
    monkeypatch.setenv("SPVAR_PT_GROUPS", str(groups))
    monkeypatch.setenv("SPVAR_PT_SPIN", str(spin))
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0, K)
    kw = dict(seed=61, icm=icm)
    got = spv.spv_pt_sample(ctx, P, betas, runs, chains, 40, **kw)
    want = oracle.pt_sample(inst, betas, runs, chains, 40, threads=8, **kw)
    _check(got, want)
    more = oracle.pt_sample(inst, betas, runs, chains, 25, sweep_offset=40, resume=want, threads=8, **kw)
    for in_place in (False, True):
        res = spv.spv_pt_sample(ctx, P, betas, runs, chains, 25, sweep_offset=40, resume=got, in_place=in_place, **kw)
        _check(res, more)


def test_beside_another_stream(spv, ctx):  # noqa: F811
    import torch
    inst = GAUSS(24)
    other = spv.Context(0)
    big = spv.Problem.from_instance(si.chimera(8, seed=3))
    P = spv.Problem.from_instance(inst)
    betas = si.geometric_betas(0.2, 5.0, 26)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        spv.spv_sample(other, big, si.linear_betas(0.1, 5.0, 1000), 10000, 3, stream=stream)
    got = spv.spv_pt_sample(ctx, P, betas, 8, 2, 60, seed=9, icm=(0, 26))
    want = oracle.pt_sample(inst, betas, 8, 2, 60, seed=9, icm=(0, 26), threads=8)
    _check(got, want)
    assert (got["top_count"].cpu().numpy() >= 0).all()
    stream.synchronize()
