"""GPU parity of the general sampler bodies' local fields at the edges of their arithmetic, bit
for bit against the oracle: every record count around the straight-line variant (odd and even, 1
to 9, and the largest, 64), couplings of +-32767, the largest field that still keeps the scaled
form (2^18 - 1) and the smallest that does not, one digit past the byte-parallel body's range, and
slice couplings on both sides of 16 bits; instance in LDS, in global memory and in a batch."""
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


def _complete_bipartite(d, j_max, x_bound, seed, scale_log2):
    """K_{d,d}: every variable has d records; couplings uniform on +-[1, j_max] with both extremes
    present, and the first variable's bias brings its |h| + sum |J| to x_bound (0: no biases)."""
    rng = np.random.default_rng(seed)
    ei, ej = np.repeat(np.arange(d), d), d + np.tile(np.arange(d), d)
    w = rng.integers(1, j_max + 1, d * d) * rng.choice([-1, 1], d * d)
    w[0], w[-1] = -j_max, j_max
    h = np.zeros(2 * d, np.int64)
    if x_bound:
        h[:] = rng.integers(-j_max, j_max + 1, 2 * d)
        h[0] = -(x_bound - np.abs(w[:d]).sum())
        for i in range(1, 2 * d):  # no other variable above the bound
            s = np.abs(w[i * d:(i + 1) * d]).sum() if i < d else np.abs(w[i - d::d]).sum()
            h[i] = np.sign(h[i]) * min(abs(h[i]), x_bound - s)
    return si.from_edges(2 * d, ei, ej, w, h, np.arange(2 * d) >= d, 2, scale_log2)


CASES = ([(f"degree{d}", d, 32767, 0, 14) for d in (1, 2, 3, 4, 5, 6, 7, 8, 9, 64)] +
         [("two_digits_largest", 6, 32767, 2 ** 18 - 1, 14), ("three_digits_smallest", 6, 32767, 2 ** 18, 14),
          ("one_digit_general", 6, 40, 511, 4), ("one_digit_general_odd", 5, 40, 256, 4)])


@pytest.mark.parametrize("name,d,j,xb,scale", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("where", ["lds", "global", "batch"])
def test_fields(spv, ctx, monkeypatch, name, d, j, xb, scale, where):
    inst = _complete_bipartite(d, j, xb, 31 + d, scale)
    if xb:
        assert oracle.x_max(inst) == xb
    betas = si.linear_betas(0.02, 2.0, 25)
    P = spv.Problem.from_instance(inst)
    print(f"[fields] {name} {where}", flush=True)
    osp, oE = oracle.sa_sample(inst, betas, reads=11, seed=5)
    if where == "batch":
        sp, E = spv.spv_sample_batch(ctx, [P, P], betas, [11, 11], [5, 5])
        sp, E = sp[1], E[1]
    else:
        monkeypatch.setenv("SPVAR_SA_BIG", "1" if where == "global" else "0")
        sp, E = spv.spv_sample(ctx, P, betas, 11, 5)
    assert np.array_equal(sp.cpu().numpy(), osp) and np.array_equal(E.cpu().numpy(), oE)


@pytest.mark.parametrize("d", [5, 6])
@pytest.mark.parametrize("gamma", [2.0, 0.02])
@pytest.mark.parametrize("big", ["0", "1"])
def test_slice_coupling_sides(spv, ctx, monkeypatch, d, gamma, big):
    """Jp crosses 32767 (the 16-bit pair) inside the two-digit range, and inside the three-digit one."""
    monkeypatch.setenv("SPVAR_SQA_BIG", big)
    inst = _complete_bipartite(d, 900, 0, 7 + d, 11)
    betas = si.linear_betas(0.3, 0.4, 16)
    gammas = np.geomspace(20.0, gamma, 16)
    jp = [oracle.sqa_coupling(b, g, 8, 11) for b, g in zip(betas, gammas)]
    assert min(jp) < 32767 < max(jp)
    print(f"[fields] sqa d={d} gamma={gamma} jp {min(jp)}..{max(jp)}", flush=True)
    sp, E = spv.spv_sqa_sample(ctx, spv.Problem.from_instance(inst), betas, gammas, 8, 6, 9)
    osp, oE, _ = oracle.sqa_sample(inst, betas, gammas, 8, reads=6, seed=9)
    assert np.array_equal(sp.cpu().numpy(), osp) and np.array_equal(E.cpu().numpy(), oE)
