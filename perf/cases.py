"""Measured cases of the framework's public entry points.

Each case is a dict of plain values; `prepare` makes what a user's program holds before the call
(a context, device problems, schedules, samples) from a seed alone, and `run` is one pass through
the binding.  Sizes are those of the repository's own workloads (periodic cubes of L = 4, 10, 20,
Chimera 8 x 8, residuals of 50 to 1000 variables) and generic ones between and around them.
"""
import math

import numpy as np
import torch

import paper_1706_07826_amd as spv


# ----------------------------------------------------------------------------- cases
def listed():
    return [
        # The smallest sampling call: L = 4 spin glass, 100 reads; the call and its 1000 dependent
        # sweeps are all latency.
        dict(name="sa_cubic4", kind="sa", graph="cubic", L=4, dist="pm1", reads=100, sweeps=1000,
             beta0=0.1, beta1=3.0, init=False),
        # The Chimera workload's full fixing sample: one launch that fills the device.
        dict(name="sa_chimera8", kind="sa", graph="chimera", L=8, dist="u6", reads=10000, sweeps=2000,
             beta0=0.1, beta1=5.0, init=False),
        # A Gaussian (two-digit) cube with the reads of a solving sample.
        dict(name="sa_cubic10", kind="sa", graph="cubic", L=10, dist="gauss", reads=1000, sweeps=1000,
             beta0=0.1, beta1=5.0, init=False),
        # A large Gaussian cube continued from caller states (resume), ragged read count.
        dict(name="sa_cubic20_resume", kind="sa", graph="cubic", L=20, dist="gauss", reads=498, sweeps=200,
             beta0=1.0, beta1=5.0, init=True),
        # Quantum annealing of the Chimera workload, 16 slices.
        dict(name="sqa_chimera8", kind="sqa", graph="chimera", L=8, dist="u6", trotter=16, reads=1000, sweeps=500),
        # Tempering over a full device: 64 runs of the L = 10 cube.
        dict(name="pt_cubic10", kind="pt", L=10, dist="gauss", K=32, runs=64, chains=1, icm=False, sweeps=1000),
        # A few short tempering runs of a small cube, on a ladder that is no multiple of four.
        dict(name="pt_cubic6_k26", kind="pt", L=6, dist="gauss", K=26, runs=8, chains=2, icm=True, sweeps=300),
        # One run of the L = 20 cube with cluster moves: 40 slots, two chains.
        dict(name="pticm_cubic20", kind="pt", L=20, dist="gauss", K=40, runs=1, chains=2, icm=True, sweeps=300),
        # The residual problems of many starts in one batched launch.
        dict(name="batch_residuals", kind="batch", graph="chimera", L=16, dist="u6", B=256, n_min=50, n_max=1000,
             reads=500, sweeps=1000),
        # Persistence over the Chimera workload's sample, and the reduced problem.
        dict(name="fix_chimera8", kind="fix", graph="chimera", L=8, dist="u6", reads=10000, elite=0.05, theta=0.95,
             gauge=2),
        # Energies of given states (another sampler's, or a merged sample's).
        dict(name="energy_cubic10", kind="energy", graph="cubic", L=10, dist="gauss", reads=10000),
        # A whole multi-start call: fixing samples, persistence, batched solving samples, recombination.
        dict(name="multistart_chimera8", kind="multistart", L=8, dist="u6", starts=20, fixing=500, solving=500,
             sweeps=1000, merge=True),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sa", "sa", "sa", "sqa", "pt", "pt", "batch", "fix", "energy", "multistart"])
    if kind in ("sa", "fix", "energy"):
        graph = rng.choice(["cubic", "chimera"])
        c = dict(kind=kind, graph=graph, L=rng.randint(4, 20) if graph == "cubic" else rng.randint(2, 16),
                 dist=rng.choice(["pm1", "gauss"]) if graph == "cubic" else "u6")
        n = _size(c)
        if kind == "sa":
            c["sweeps"] = _logint(rng, 50, 2000)
            cap = 8e9 if c["dist"] != "gauss" else 2e9
            c["reads"] = max(5, min(_logint(rng, 10, 10000), int(cap / n / c["sweeps"])))
            c.update(beta0=0.1, beta1=rng.choice([3.0, 5.0]), init=rng.random() < 0.25)
        else:
            c["reads"] = min(_logint(rng, 500 if kind == "fix" else 50, 10000), 20_000_000 // n)
            if kind == "fix":
                c.update(elite=rng.choice([0.05, 0.1, 0.2]), theta=rng.choice([0.9, 0.95, 1.0]),
                         gauge=rng.randint(0, 2))
        return c
    if kind == "sqa":
        c = dict(kind=kind, graph="chimera", L=rng.randint(3, 8), dist="u6", trotter=rng.choice([8, 16, 24, 32]),
                 sweeps=_logint(rng, 50, 500))
        c["reads"] = max(5, min(_logint(rng, 20, 1000), int(4e9 / (_size(c) * c["trotter"] * c["sweeps"]))))
        return c
    if kind == "pt":
        L = rng.randint(4, 20)
        if L > 10:
            return dict(kind=kind, L=L, dist="gauss", K=4 * rng.randint(4, 10), runs=1, chains=2, icm=True,
                        sweeps=_logint(rng, 50, 300))
        chains = rng.randint(1, 2)
        return dict(kind=kind, L=L, dist=rng.choice(["gauss", "pm1"]),
                    K=rng.randint(8, 30) if L <= 7 else 4 * rng.randint(4, 8), runs=_logint(rng, 1, 32),
                    chains=chains, icm=chains == 2 and rng.random() < 0.7, sweeps=_logint(rng, 100, 1000))
    if kind == "batch":
        graph = rng.choice(["chimera", "cubic"])
        return dict(kind=kind, graph=graph, L=16 if graph == "chimera" else 12,
                    dist="u6" if graph == "chimera" else "gauss", B=_logint(rng, 8, 128), n_min=rng.randint(30, 80),
                    n_max=rng.randint(300, 1000), reads=_logint(rng, 50, 500), sweeps=_logint(rng, 100, 1000))
    return dict(kind="multistart", L=rng.randint(4, 8), dist="u6", starts=rng.randint(4, 20),
                fixing=_logint(rng, 50, 500), solving=_logint(rng, 50, 500), sweeps=_logint(rng, 100, 1000),
                merge=rng.random() < 0.5)


def _size(c):
    return 8 * c["L"] ** 2 if c.get("graph") == "chimera" or c["kind"] == "multistart" else c["L"] ** 3


# ----------------------------------------------------------------------------- inputs
def _edges(graph, L):
    """Undirected edges (i, j) of a periodic L^3 cube or an L x L Chimera graph, and a 2-colouring
    (None where the cube's odd side has none)."""
    if graph == "cubic":
        i = np.arange(L ** 3)
        x, y, z = i % L, (i // L) % L, i // (L * L)
        j = np.stack([(x + 1) % L + L * (y + L * z), x + L * ((y + 1) % L + L * z), x + L * (y + L * ((z + 1) % L))], 1)
        return np.repeat(i, 3), j.reshape(-1), None if L % 2 else (x + y + z) & 1
    cell = np.arange(L * L)
    a, b = np.meshgrid(np.arange(4), np.arange(4), indexing="ij")
    ei = [(8 * cell[:, None] + a.reshape(1, -1)).reshape(-1)]
    ej = [(8 * cell[:, None] + 4 + b.reshape(1, -1)).reshape(-1)]
    r, c = cell // L, cell % L
    u = np.arange(4)
    down, right = cell[r < L - 1], cell[c < L - 1]
    ei += [(8 * down[:, None] + u).reshape(-1), (8 * right[:, None] + 4 + u).reshape(-1)]
    ej += [(8 * (down[:, None] + L) + u).reshape(-1), (8 * (right[:, None] + 1) + 4 + u).reshape(-1)]
    i = np.arange(8 * L * L)
    cl = i // 8
    return np.concatenate(ei), np.concatenate(ej), ((i % 8) >> 2) ^ ((cl // L + cl % L) & 1)


def _first_fit(n, rp, col):
    """First-fit colour classes in index order (odd periodic cubes: three or four classes)."""
    colour = np.full(n, -1)
    for i in range(n):
        used = set(colour[col[rp[i]:rp[i + 1]]].tolist())
        k = 0
        while k in used:
            k += 1
        colour[i] = k
    return colour


def _csr(n, ei, ej, w):
    a, b, v = np.concatenate([ei, ej]), np.concatenate([ej, ei]), np.concatenate([w, w])
    o = np.lexsort((b, a))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(a, minlength=n), out=rp[1:])
    return rp, b[o], v[o]


def _instance(graph, L, dist, rng):
    """(n, row_ptr, col, J, h, colour, n_colours, scale_log2) on the host: +-1 or Gaussian x 2^10
    couplers without biases, or couplers and biases uniform on +-1..6."""
    ei, ej, colour = _edges(graph, L)
    n = 8 * L * L if graph == "chimera" else L ** 3
    h = np.zeros(n, np.int64)
    scale = 0
    if dist == "pm1":
        w = rng.choice([-1, 1], ei.size)
    elif dist == "gauss":
        w = np.clip(np.rint(rng.standard_normal(ei.size) * 1024), -32767, 32767).astype(np.int64)
        scale = 10
    else:
        vals = np.array([k for k in range(-6, 7) if k])
        w, h = rng.choice(vals, ei.size), rng.choice(vals, n)
    rp, col, J = _csr(n, ei, ej, w)
    if colour is None:
        colour = _first_fit(n, rp, col)
    return n, rp, col, J, h, colour, int(colour.max()) + 1, scale


def _residuals(c, rng):
    """Breadth-first balls of a parent instance, n log-uniform, the rest frozen at a random state
    and folded into the biases."""
    n, rp, col, J, h, colour, nc, scale = _instance(c["graph"], c["L"], c["dist"], rng)
    nbr = [col[rp[i]:rp[i + 1]].tolist() for i in range(n)]
    rows = np.repeat(np.arange(n), np.diff(rp))
    out = []
    # (the sizes are the same for every seed: evenly spread quantiles of the log-uniform law)
    q = (np.arange(c["B"]) + 0.5) / c["B"]
    for size in np.exp(math.log(c["n_min"]) + q * math.log(c["n_max"] / c["n_min"])).astype(int):
        root = int(rng.integers(n))
        seen, todo = {root}, [root]
        for i in todo:
            if len(todo) >= size:
                break
            for j in nbr[i]:
                if j not in seen:
                    seen.add(j)
                    todo.append(j)
        keep = np.sort(np.array(todo[:size]))
        inside = np.zeros(n, bool)
        inside[keep] = True
        s = rng.choice([-1, 1], n)
        hk = h + np.bincount(rows, weights=J * s[col] * ~inside[col], minlength=n).astype(np.int64)
        new = np.cumsum(inside) - 1
        e = inside[rows] & inside[col]
        r2 = np.zeros(keep.size + 1, np.int64)
        np.cumsum(np.bincount(new[rows[e]], minlength=keep.size), out=r2[1:])
        out.append((keep.size, r2, new[col[e]], J[e], hk[keep], colour[keep], nc, scale))
    return out


def _device(inst):
    n, rp, col, J, h, colour, nc, scale = inst
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a, dt)).cuda()
    return spv.Problem(n, int(rp[-1]), t(rp, np.int32), t(col, np.int32), t(J, np.int32), t(h, np.int32),
                       t(colour, np.uint8), nc, scale)


def _energies(inst, S):
    """E of the rows of S (int8 [R][n], any device) in 64-bit integers."""
    n, rp, col, J, h = inst[:5]
    rows = np.repeat(np.arange(n), np.diff(rp))
    up = rows < col
    t = lambda a: torch.as_tensor(np.asarray(a, np.int64), device=S.device)
    ei, ej, w, hh = t(rows[up]), t(col[up]), t(J[up]), t(h)
    E = torch.empty(S.shape[0], dtype=torch.int64, device=S.device)
    step = max(1, 40_000_000 // max(1, ei.numel()))
    for a in range(0, S.shape[0], step):
        s = S[a:a + step].long()
        E[a:a + step] = (s[:, ei] * s[:, ej] * w).sum(1) + (s * hh).sum(1)
    return E


def _sample(n, reads, rng):
    """A sample as an annealer leaves it: 60 % of the variables agree in every read, the rest vary.
    (Which ones is the same for every seed, so a reduced problem has the same sizes.)"""
    base = rng.choice([-1, 1], n).astype(np.int8)
    p = np.where(np.random.default_rng(n).random(n) < 0.6, 0.0, 0.2 + 0.3 * rng.random(n)).astype(np.float32)
    return np.where(rng.random((reads, n), dtype=np.float32) < p, -base, base).astype(np.int8)


def _fix_inputs(c, seed):
    rng = np.random.default_rng(seed)
    inst = _instance(c["graph"], c["L"], c["dist"], rng)
    return inst, _sample(inst[0], c["reads"], rng)


# ----------------------------------------------------------------------------- passes
def prepare(c, seed):
    st = dict(case=c, ctx=spv.spv_ctx_create(torch.cuda.current_device()), seed=int(seed) * 7919 + 1)
    kind = c["kind"]
    if kind in ("fix", "energy"):
        inst, S = _fix_inputs(c, seed)
        st["S"] = torch.as_tensor(S).cuda()
        st["P"] = _device(inst)
        if kind == "fix":
            st["E"] = _energies(inst, st["S"])
        return st
    rng = np.random.default_rng(seed)
    if kind == "batch":
        st["P"] = [_device(i) for i in _residuals(c, rng)]
        st["betas"] = np.linspace(0.1, 5.0, c["sweeps"])
        st["seeds"] = [st["seed"] + b for b in range(c["B"])]
        # one buffer of every instance's reads, and its views
        sizes = [c["reads"] * p.n for p in st["P"]]
        st["spins"] = torch.empty(sum(sizes), dtype=torch.int8, device="cuda")
        st["energies"] = torch.empty((c["B"], c["reads"]), dtype=torch.int64, device="cuda")
        st["spin_views"] = [v.view(c["reads"], -1) for v in st["spins"].split(sizes)]
        st["energy_views"] = list(st["energies"])
        return st
    graph = "chimera" if kind == "multistart" else c.get("graph", "cubic")
    inst = _instance(graph, c["L"], c["dist"], rng)
    st["P"] = _device(inst)
    if kind == "sa":
        st["betas"] = np.linspace(c["beta0"], c["beta1"], c["sweeps"])
        if c["init"]:
            st["init"] = torch.as_tensor(_sample(inst[0], c["reads"], rng)).cuda()
    elif kind == "sqa":
        st["betas"] = np.linspace(0.1, 5.0, c["sweeps"])
        st["gammas"] = np.geomspace(3.0, 0.01, c["sweeps"])
    elif kind == "pt":
        st["betas"] = np.geomspace(0.2, 5.0, c["K"])
    else:
        st["betas"] = np.linspace(0.1, 5.0, c["sweeps"])
    return st


def run(st):
    c, ctx, P, seed = st["case"], st["ctx"], st["P"], st["seed"]
    kind = c["kind"]
    if kind == "sa":
        return spv.spv_sample(ctx, P, st["betas"], c["reads"], seed, sweep_offset=1000 if c["init"] else 0,
                              init_spins=st.get("init"))
    if kind == "sqa":
        return spv.spv_sqa_sample(ctx, P, st["betas"], st["gammas"], c["trotter"], c["reads"], seed)
    if kind == "pt":
        return spv.spv_pt_sample(ctx, P, st["betas"], c["runs"], c["chains"], c["sweeps"], seed,
                                 icm=(0, c["K"]) if c["icm"] else None)
    if kind == "batch":
        spv.spv_sample_batch(ctx, P, st["betas"], [c["reads"]] * c["B"], st["seeds"], spins=st["spin_views"],
                             energies=st["energy_views"], graph=True)
        return dict(spins=st["spins"], energies=st["energies"])
    if kind == "fix":
        fx = spv.spv_persist_fix(ctx, P, st["S"], st["E"], c["elite"], c["theta"], gauge=c["gauge"])
        i, Q = fx.info(), fx.reduced()  # the next stage needs the reduced sizes
        k = fx.orig_index
        return dict(mask=fx.fixed_mask, val=fx.fixed_val, orig=k, row_ptr=Q.row_ptr, col=Q.col[:Q.nnz],
                    J=Q.J[:Q.nnz], h=Q.h[:Q.n], colour=Q.colour[:Q.n], offset=i["offset"], m=i["m"],
                    k_min=i["k_min"], pivot=i["pivot"])
    if kind == "energy":
        return spv.spv_energy(ctx, P, st["S"])
    return spv.spv_multistart(ctx, P, st["betas"], seed, c["starts"], c["fixing"], c["solving"], 0.2, 1.0,
                              gauge=0, merge=c["merge"])


# ----------------------------------------------------------------------------- work and exact values
def _ops(updates, degree, digits):
    """Integer operations of Metropolis updates: per digit a quarter of a Philox4x32-10 block (four
    words serve four replicas; 20 products, 20 three-input xors), a multiply-add per neighbour, and
    sign, digit, comparison and flip."""
    return updates * (10 * digits + 2 * degree + 4)


def work(c):
    kind, n = c["kind"], _size(c)
    deg = 6
    problem = n * (4 + 4 + 1) + n * deg * 8
    dig = 2 if c["dist"] == "gauss" else 1
    if kind == "sa":
        out = c["reads"] * (n + 8)
        return dict(bytes=problem + out + (c["reads"] * n if c["init"] else 0),
                    flops=_ops(n * c["reads"] * c["sweeps"], deg, dig))
    if kind == "sqa":
        return dict(bytes=problem + c["reads"] * (n + 8),
                    flops=_ops(n * c["trotter"] * c["reads"] * c["sweeps"], deg + 2, 1))
    if kind == "pt":
        reps = c["runs"] * c["chains"] * c["K"]
        return dict(bytes=problem + reps * (n + 8) + reps // 2 * 10 * (n + 8),
                    flops=_ops(n * reps * c["sweeps"], deg, dig))
    if kind == "batch":
        mean = (c["n_max"] - c["n_min"]) / math.log(c["n_max"] / c["n_min"])
        return dict(bytes=int(c["B"] * mean * (9 + deg * 8 + c["reads"])),
                    flops=_ops(int(c["B"] * mean) * c["reads"] * c["sweeps"], deg, dig))
    if kind == "fix":
        elite = max(1, math.ceil(c["elite"] * c["reads"]))
        return dict(bytes=2 * problem + 8 * c["reads"] + elite * n, flops=elite * n)
    if kind == "energy":
        return dict(bytes=problem + c["reads"] * (n + 8), flops=c["reads"] * n * (deg + 1))
    reads = c["starts"] * (c["fixing"] + c["solving"] // 4)
    return dict(bytes=problem + c["starts"] * (8 * (c["fixing"] + c["solving"]) + 2 * n),
                flops=_ops(n * reads * c["sweeps"], deg, dig))


def exact(c, seed):
    # Sampler outputs are pseudo-random states, not computed values.  Energies of given states are exact
    # integers.  Persistence outputs are whole numbers throughout, derived by counting.
    if c["kind"] == "energy":
        inst, S = _fix_inputs(c, seed)
        return _energies(inst, torch.as_tensor(S).cuda())
    return None
