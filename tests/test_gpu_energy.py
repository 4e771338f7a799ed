"""Energies of given rows, exactly against the oracle: sizes at the edges of a workgroup and of what
the LDS holds (n = 16384, global gathers beyond), odd record counts, row
counts around the rows of a workgroup, and any int8 value in the rows."""
import numpy as np
import pytest

import oracle
import spvar_inputs as si

pytestmark = pytest.mark.gpu

CASES = ([(n, R, 6) for n, R in [(1, 1), (2, 3), (63, 4), (257, 5), (1024, 4095), (1025, 4096), (1000, 4099),
                                    (512, 1024), (512, 1025), (513, 1024)]] +
         [(4096, 9, 5), (4097, 9, 5), (8192, 4097, 3), (8193, 4097, 3), (16384, 6, 3), (16385, 6, 3),
          (130, 8193, 1), (300, 4100, 64), (200, 7, 63)])


def _ring(n, D, seed):
    """Site i joined to i + 1 .. i + D // 2 (and, for odd D, to i + n / 2) modulo n; beyond 8 records
    even sites to the D odd ones that follow."""
    rng = np.random.default_rng(seed)
    if D > 8:
        edges = {tuple(sorted((i, (i + 2 * k + 1) % n))) for k in range(D) for i in range(0, n, 2)}
    else:
        edges = {tuple(sorted((i, (i + k) % n))) for k in range(1, D // 2 + 1) for i in range(n) if (i + k) % n != i}
        if D & 1:
            edges |= {(i, i + n // 2) for i in range(n // 2)}
    e = np.array(sorted(edges), np.int64).reshape(-1, 2)
    w = rng.choice([-32767, 32767, -5, 7], len(e))
    h = rng.integers(-2 ** 25, 2 ** 25, n)
    adj = [[] for _ in range(n)]
    for a, b in e:
        adj[a].append(b)
        adj[b].append(a)
    colour = np.full(n, -1)
    for i in range(n):
        used = {colour[j] for j in adj[i]}
        colour[i] = next(k for k in range(n) if k not in used)
    return si.from_edges(n, e[:, 0], e[:, 1], w, h, colour, int(colour.max()) + 1, 0)


@pytest.mark.parametrize("n,R,D", CASES)
def test_energy(n, R, D):
    import torch
    import paper_1706_07826_amd as spv
    inst = _ring(n, D, n + D)
    rng = np.random.default_rng(R)
    ctx = spv.Context(0)
    P = spv.Problem.from_instance(inst)
    for lo, hi in ((-1, 1), (-128, 127)):
        S = rng.choice([-1, 1], (R, n)) if lo == -1 else rng.integers(lo, hi + 1, (R, n))
        S = S.astype(np.int8)
        print(f"[energy] n={n} R={R} D={D} values {lo}..{hi}", flush=True)
        E = spv.spv_energy(ctx, P, torch.as_tensor(S).cuda()).cpu().numpy()
        assert np.array_equal(E, oracle.energy(inst, S))
