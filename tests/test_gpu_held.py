"""GPU parity of the byte-parallel SA body that holds a lane's sites in registers, bit for bit
against the oracle: 3 to 8 records a site (odd counts padded), two to four colour classes, class
sizes at the edges of waves and of the largest workgroup and unequal ones, one to several quads per
workgroup, ragged reads, caller states, and the streamed launch."""
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


def _layers(sizes, d, j_max, seed, h_max=0):
    """One class per entry of `sizes`; site i of a class is joined to d consecutive sites of every
    later class (circulant), so rows have at most d records per other class."""
    rng = np.random.default_rng(seed)
    base = np.concatenate([[0], np.cumsum(sizes)])
    edges = set()
    for a in range(len(sizes)):
        for b in range(a + 1, len(sizes)):
            m = max(sizes[a], sizes[b])
            for i in range(m):
                for k in range(d):
                    edges.add((int(base[a] + i % sizes[a]), int(base[b] + (i + k) % sizes[b])))
    e = np.array(sorted(edges))
    n = int(base[-1])
    w = rng.integers(1, j_max + 1, len(e)) * rng.choice([-1, 1], len(e))
    h = rng.integers(-h_max, h_max + 1, n) if h_max else np.zeros(n, np.int64)
    return si.from_edges(n, e[:, 0], e[:, 1], w, h, np.repeat(np.arange(len(sizes)), sizes), len(sizes), 0)


CASES = ([(f"degree{d}", [40, 40], d, 6, 5, 21, {}) for d in (3, 4, 5, 6, 7, 8)] +
         [(f"class{m}", [m, m], 3, 3, 2, 13, {}) for m in (8, 9, 31, 63, 64, 65, 256, 257)] +
         [("largest", [1024, 1024], 4, 3, 0, 7, {}), ("beyond", [1025, 1025], 4, 3, 0, 7, {}),
          ("three", [50, 50, 50], 2, 4, 3, 19, {}), ("four", [40, 40, 40, 40], 2, 4, 3, 19, {}),
          ("five_not_held", [20] * 5, 1, 4, 3, 19, {}),
          ("unequal", [90, 45], 4, 5, 3, 19, {}), ("bound255", [30, 30], 5, 51, 0, 19, {}),
          ("quads5", [40, 40], 6, 6, 5, 37, {"SPVAR_SA_HELD": 5}), ("off", [40, 40], 6, 6, 5, 21, {"SPVAR_SA_HELD": 0}),
          ("stream", [40, 40], 6, 6, 5, 150, {"SPVAR_SA_STREAM": 8}),
          ("stream_four", [40, 40, 40, 40], 2, 4, 3, 150, {"SPVAR_SA_STREAM": 8})])


@pytest.mark.parametrize("init", [False, True])
@pytest.mark.parametrize("name,sizes,d,j,h,reads,env", CASES, ids=[c[0] for c in CASES])
def test_held(spv, ctx, monkeypatch, name, sizes, d, j, h, reads, env, init):
    import torch
    inst = _layers(sizes, d, j, 5 + d, h)
    assert oracle.x_max(inst) <= 255
    for k, v in env.items():
        monkeypatch.setenv(k, str(v))
    sweeps = 48 if "stream" in name else 21
    betas = np.concatenate([[0.0], si.linear_betas(0.05, 3.0, sweeps - 1)])
    S0 = si.random_spins(reads, inst.n, seed=3) if init else None
    print(f"[held] {name} n={inst.n} reads={reads} init={init}", flush=True)
    sp, E = spv.spv_sample(ctx, spv.Problem.from_instance(inst), betas, reads, 17, sweep_offset=9 if init else 0,
                           init_spins=torch.as_tensor(S0).cuda() if init else None)
    osp, oE = oracle.sa_sample(inst, betas, reads=reads, seed=17, sweep_offset=9 if init else 0, init=S0, threads=8)
    assert np.array_equal(sp.cpu().numpy(), osp) and np.array_equal(E.cpu().numpy(), oE)


BATCHES = [
    ("two_classes", [[40, 40], [9, 8], [129, 64], [300, 257], [1, 1]], 3, [23, 400, 9, 30, 3]),
    ("degree5_padded", [[30, 30], [64, 64]], 5, [50, 700]),
    ("degree8", [[30, 30], [20, 31]], 8, [50, 70]),
    ("three_classes", [[20, 20, 20], [33, 31, 35]], 2, [41, 17]),
    ("four_classes", [[20, 20, 20, 20], [65, 12, 9, 64]], 2, [41, 17]),
    ("mixed_class_counts", [[20, 20], [12, 12, 12]], 3, [41, 17]),
    ("fills_device_wide", [[300, 300], [40, 40]], 4, [8200, 900]),
    ("fills_device_narrow", [[60, 60], [40, 40]], 4, [40100, 900]),
]


@pytest.mark.parametrize("name,shapes,d,reads", BATCHES, ids=[c[0] for c in BATCHES])
def test_held_batch(spv, ctx, name, shapes, d, reads):
    insts = [_layers(sz, min(d, min(sz)), 6, 50 + b, 4) for b, sz in enumerate(shapes)]
    betas = si.linear_betas(0.05, 3.0, 11)
    seeds = [70 + b for b in range(len(insts))]
    print(f"[held] batch {name}", flush=True)
    probs = [spv.Problem.from_instance(i) for i in insts]
    for graph in (False, True, True):
        sp, E = spv.spv_sample_batch(ctx, probs, betas, reads, seeds, graph=graph)
        for b, inst in enumerate(insts):
            s_b, e_b = sp[b].cpu().numpy(), E[b].cpu().numpy()
            assert np.array_equal(e_b, oracle.energy(inst, s_b)), b
            for lo, hi in {(0, min(40, reads[b])), (max(0, reads[b] - 40), reads[b])}:
                osp, oE = oracle.sa_sample(inst, betas, seed=seeds[b], r_begin=lo, r_end=hi)
                assert np.array_equal(s_b[lo:hi], osp) and np.array_equal(e_b[lo:hi], oE), (b, lo)
