"""Performance cases of the TensorRVEA library: the work that its users run.

A case is a dict of plain values; ``prepare`` builds what a program holds before
the call, ``run`` makes one pass through the public entry points and returns its
outputs, ``work`` counts the bytes and operations that the pass cannot do
without, and ``exact`` gives the pass's outputs in 64 bits by plain torch.

Kinds of case:

evolve      a run handle kept by the program: some generations, then the
            objectives of the population (monitoring a run in progress)
job         a whole optimisation: create a run in a kept workspace, all its
            generations, the final population with its genes, close
generation  a population held on the host (a checkpoint, or another process's
            individuals) loaded into a run, one generation, the result read back
policy      evolve on the policy-rollout problem (neuroevolution)
batch       independent runs advanced together, then every run's objectives
indicators  hypervolume and expected utility of a population on the device
"""
import math

import numpy as np
import torch

import paper_2404_01159_amd as P

DEV = "cuda:0"
ROLLOUTS, STEPS = 16, 200  # per policy, as the policy workload of the benchmark
SITES = 32  # mutation sites that a child can hold


# ------------------------------------------------------------------ the cases
def lattice(m, n):
    """(H, K) of the smallest Das-Dennis lattice with at least n vectors."""
    h = 1
    while math.comb(h + m - 1, m - 1) < n:
        h += 1
    return h, math.comb(h + m - 1, m - 1)


def evolve(name, problem, m, n, d, gens, op="ga", kind="evolve"):
    case = dict(kind=kind, problem=problem, m=m, n=n, d=d, gens=gens, op=op)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one small optimisation from start to end, as an application makes many of them
        evolve("job_m3_n105_d12", 2, 3, 105, 12, 100, kind="job"),
        # the smallest population of the scaling study: latency of the generation loop
        evolve("evolve_m3_n32_d100", 1, 3, 32, 100, 50),
        # the middle of the scaling study; more vectors than individuals (2,080)
        evolve("evolve_m3_n2048_d100", 1, 3, 2048, 100, 20),
        # the benchmark's default workload
        evolve("evolve_m3_n10011_d500", 1, 3, 10011, 500, 20),
        # the largest population and gene pool (4 GB)
        evolve("evolve_m3_n100128_d5000", 3, 3, 100128, 5000, 10),
        # few individuals with very long rows (second scaling study)
        evolve("evolve_m3_n100_d131072", 1, 3, 100, 131072, 20),
        # many objectives: no index of the vectors, odd sizes
        evolve("evolve_m5_n3876_d301", 3, 5, 3876, 301, 10),
        # two objectives and a swarm operator (velocities beside the genes)
        evolve("evolve_m2_n5000_d700_pso", 2, 2, 5000, 700, 10, op="pso"),
        # a checkpoint resumed, advanced and saved: host data both ways
        evolve("generation_m3_n2016_d1000", 1, 3, 2016, 1000, 1, kind="generation"),
        # neuroevolution: 4,096 policy networks by rollouts on the matrix cores
        dict(name="policy_n4096", kind="policy", n=4096, gens=2, op="ga"),
        # sixteen runs of the serving mix (m = 2, 3, 5, 8), one submission per generation
        dict(name="batch_16", kind="batch", runs=16, mix=1, gens=10),
        # quality of a final population of the benchmark's default workload
        dict(name="indicators_m3_n10011_w5151", kind="indicators", m=3, n=10011, weights=5151),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve"] * 5 + ["job", "generation", "policy", "batch", "indicators"])
    ops = ["ga"] * 5 + ["de", "pso", "cso", "rand"]
    if kind == "evolve":
        if rng.random() < 0.2:  # long rows, few individuals
            return evolve(None, rng.randint(1, 3), 3, rng.randint(50, 200), log_int(rng, 512, 262144),
                          rng.choice([10, 20]))
        m = rng.choice([2, 3, 3, 3, 5, 8])
        n = log_int(rng, 32, 20000 if m <= 3 else 6000)
        return evolve(None, rng.randint(1, 3), m, n, log_int(rng, 12, min(5000, 40_000_000 // n)),
                      rng.choice([10, 20]), rng.choice(ops))
    if kind == "job":
        n = log_int(rng, 32, 1000)
        return evolve(None, rng.randint(1, 3), rng.choice([2, 3, 4]), n, log_int(rng, 12, 500),
                      rng.choice([50, 100]), rng.choice(ops), kind="job")
    if kind == "generation":
        n = log_int(rng, 64, 4000)
        return evolve(None, rng.randint(1, 3), rng.choice([2, 3, 3, 5]), n,
                      log_int(rng, 30, min(3000, 4_000_000 // n)), 1, rng.choice(ops),
                      kind="generation")
    if kind == "policy":
        return dict(kind="policy", n=log_int(rng, 64, 4096), gens=rng.randint(1, 3),
                    op=rng.choice(ops))
    if kind == "batch":
        return dict(kind="batch", runs=rng.randint(3, 24), mix=rng.randint(2, 1000), gens=10)
    m = rng.choice([2, 3, 3])
    return dict(kind="indicators", m=m, n=log_int(rng, 50, 16000),
                weights=lattice(m, log_int(rng, 50, 6000))[1])


# ------------------------------------------------------------- what a pass needs
def params_of(case, **more):
    """Run parameters: an adaptation every ten generations, as in a run of 100."""
    return P.default_params(case.get("op", "ga"), t_max=100, **more)


def lq_system(seed):
    """A seeded stable linear system for the policies to steer."""
    r = np.random.default_rng(seed)
    g = r.standard_normal((32, 32))
    a = 0.95 * g / np.max(np.abs(np.linalg.eigvals(g)))
    return dict(A=a.astype(np.float32), B=(0.1 * r.standard_normal((32, 8))).astype(np.float32),
                x0=r.standard_normal((ROLLOUTS, 32)).astype(np.float32), T=STEPS, sigma=0.1)


def serving_mix(case):
    """Shapes of a batch's runs: objectives, genes and lattice as the served requests have."""
    r = np.random.default_rng(case["mix"])
    spans = {2: (99, 10010), 3: (13, 140), 5: (5, 19), 8: (3, 8)}
    out = []
    for _ in range(case["runs"]):
        m = int(r.choice([2, 3, 5, 8]))
        h = int(r.integers(spans[m][0], spans[m][1] + 1))
        out.append(dict(problem=int(r.integers(1, 4)), m=m, d=int(r.integers(30, 2001)),
                        K=math.comb(h + m - 1, m - 1)))
    return out


def shape(case):
    """(n, d, m, K) of an evolving population."""
    if case["kind"] == "policy":
        return case["n"], P.POLICY_D, 2, max(case["n"], 2)
    return case["n"], case["d"], case["m"], lattice(case["m"], case["n"])[1]


def weight_lattice(m, k):
    """The k simplex weights of the lattice with that many, k x m doubles."""
    h, _ = lattice(m, k)
    grid = np.stack(np.meshgrid(*[np.arange(h + 1)] * (m - 1), indexing="ij"), -1).reshape(-1, m - 1)
    grid = grid[grid.sum(1) <= h]
    return np.concatenate([grid, h - grid.sum(1, keepdims=True)], 1) / h


def front(case, seed):
    """Objectives near a spherical front and the survivors' mask (one slot in eight is empty)."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, m = case["n"], case["m"]
    w = torch.empty(n, m, device=DEV, dtype=torch.float64).exponential_(generator=g)
    r = 1.0 + 0.05 * torch.rand(n, 1, device=DEV, dtype=torch.float64, generator=g)
    f = (r * w / w.norm(dim=1, keepdim=True)).float()
    valid = (torch.rand(n, device=DEV, generator=g) < 0.875).to(torch.uint8)
    valid[0] = 1
    return f, valid


def host_population(case, seed):
    """Uniform genes, their objectives (in 64 bits, stored in 32), all individuals present."""
    n, d, m, K = shape(case)
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.zeros(K, d, device=DEV)
    x[:n] = torch.rand(n, d, device=DEV, generator=g)
    f = torch.full((K, m), math.nan, device=DEV)
    f[:n] = objectives(case["problem"], m, x[:n].double()).float()
    valid = np.zeros(K, np.uint8)
    valid[:n] = 1
    return x.cpu().numpy(), f.cpu().numpy(), valid


def prepare(case, seed):
    kind = case["kind"]
    if kind == "indicators":
        f, valid = front(case, seed)
        w = torch.from_numpy(weight_lattice(case["m"], case["weights"])).to(DEV)
        return dict(kind=kind, F=f, valid=valid, W=w, lo=[0.0] * case["m"], hi=[1.1] * case["m"])
    if kind == "batch":
        batch = P.Batch(case["runs"], device=DEV)
        for i, s in enumerate(serving_mix(case)):
            batch.admit(P.Run(s["problem"], s["m"], s["d"], s["K"], s["K"], seed=1000 * seed + i,
                              params=params_of(case), device=DEV))
        return dict(kind=kind, batch=batch, gens=case["gens"])
    n, d, m, K = shape(case)
    if kind == "policy":
        run = P.Run(P.POLICY_LQ, 2, d, n, K, seed=seed, params=params_of(case, lb=-1.0, ub=1.0),
                    device=DEV, system=lq_system(seed))
        run.prepare(case["gens"])
        return dict(kind=kind, run=run, gens=case["gens"])
    prm = params_of(case)
    if kind == "job":
        ws = torch.empty(P.footprint(case["problem"], m, d, n, K, prm) + 256, dtype=torch.uint8,
                         device=DEV)
        return dict(kind=kind, case=dict(case), shape=(n, d, m, K), seed=seed, params=prm, ws=ws)
    run = P.Run(case["problem"], m, d, n, K, seed=seed, params=prm, device=DEV)
    run.prepare(case["gens"])  # the program's loop calls it with the same count each time
    state = dict(kind=kind, run=run, gens=case["gens"])
    if kind == "generation":
        state["X"], state["F"], state["valid"] = host_population(case, seed)
    return state


def run(state):
    kind = state["kind"]
    if kind == "indicators":
        hv = P.hypervolume(state["F"], state["valid"], state["lo"], state["hi"])
        eu = P.expected_utility(state["F"], state["W"], state["valid"], state["lo"], state["hi"])
        return dict(hypervolume=hv, expected_utility=eu)
    if kind == "batch":
        state["batch"].step(state["gens"])
        out = []
        for r in state["batch"].runs:
            s = r.get_state(genes=False)
            out.append((s["F"], s["valid"]))
        return out
    if kind == "job":
        n, d, m, K = state["shape"]
        job = P.Run(state["case"]["problem"], m, d, n, K, seed=state["seed"],
                    params=state["params"], device=DEV, workspace=state["ws"])
        job.run(state["case"]["gens"])
        out = job.get_state()
        job.close()
        return out
    r = state["run"]
    if kind == "generation":
        r.set_state(state["X"], state["F"], state["valid"])
        r.run(1)
        return r.get_state()
    r.run(state["gens"])
    return r.get_state(genes=False)


# ------------------------------------------------------------------------ work
def generation_work(n, d, m, K, op):
    """Bytes and operations of one generation: the parents' genes read and the children's written
    (swarms: velocities too), every merged row's objectives and association, every vector once; about
    fifty operations per child gene (random bits, spread factor, child, distance term)."""
    rows = {"ga": 2, "de": 2, "pso": 4, "cso": 4, "rand": 1}[op]
    return 4.0 * rows * n * d + (4 * m + 21) * (n + K) + 8 * m * K, 50.0 * n * d


def work(case):
    kind = case["kind"]
    if kind == "indicators":
        n, m = case["n"], case["m"]
        return dict(bytes=4 * n * m + n + 8 * m * case["weights"],
                    flops=20.0 * n * math.log2(n + 1) + 2.0 * m * n * case["weights"])
    if kind == "batch":
        parts = [generation_work(s["K"], s["d"], s["m"], s["K"], "ga") for s in serving_mix(case)]
        return dict(bytes=case["gens"] * sum(b for b, _ in parts),
                    flops=case["gens"] * sum(f for _, f in parts))
    n, d, m, K = shape(case)
    b, f = generation_work(n, d, m, K, case["op"])
    if kind == "policy":
        per_step = 2 * (64 * 32 + 64 * 64 + 8 * 64) + 2 * (32 * 32 + 32 * 8)
        f += float(per_step) * n * ROLLOUTS * STEPS
    moved = 4.0 * K * d * (2 if kind == "generation" else 1 if kind == "job" else 0)
    return dict(bytes=case["gens"] * b + moved, flops=case["gens"] * f)


# ----------------------------------------------------------- outputs in 64 bits
M32 = 0xFFFFFFFF


def philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 of broadcastable int64 counter words; four int64 words."""
    k0, k1 = seed & M32, (seed >> 32) & M32
    c0, c1, c2, c3 = torch.broadcast_tensors(*[torch.as_tensor(c, device=DEV) for c in (c0, c1, c2, c3)])
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((b >> 32) & M32) ^ c1 ^ k0, b & M32, ((a >> 32) & M32) ^ c3 ^ k1, a & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def gene_words(units, d, t, tag, seed):
    """One word per gene: word g % 4 of counter (g / 4, unit, t, tag); units x d."""
    q = torch.arange((d + 3) // 4, device=DEV)
    w = philox(q[None, :], torch.arange(units, device=DEV)[:, None], t, tag, seed)
    return torch.stack(w, -1).reshape(units, -1)[:, :d]


def u24(w):
    return (w >> 8).double() * 2.0 ** -24


def u53(a, b):
    return (((a >> 5) << 26) | (b >> 6)).double() * 2.0 ** -53


def objectives(problem, m, x):
    """Objectives of genes x (n x d, 64 bits) of the test problems."""
    y = torch.sort(x[:, :m - 1], dim=1).values
    w = torch.diff(y, dim=1, prepend=torch.zeros_like(y[:, :1]), append=torch.ones_like(y[:, :1]))
    t = x[:, m - 1:] - 0.5
    if problem == 2:
        g = 4 * (t * t).mean(1)
    else:
        g = (10 * t * t + 2 * torch.sin(4 * math.pi * t) ** 2).mean(1)
    if problem != 1:
        w = w / w.norm(dim=1, keepdim=True)
    return (1 + g)[:, None] * w


def simplex_vectors(m, K):
    w = torch.from_numpy(weight_lattice(m, K)).to(DEV)
    return w / w.norm(dim=1, keepdim=True)


def nearest(rows, v, skip_self=False):
    """Largest cosine of each row with the unit vectors v, and its vector."""
    best, arg = [], []
    for s in range(0, len(rows), 2048):
        c = rows[s:s + 2048] @ v.T
        if skip_self:
            i = torch.arange(len(c), device=DEV)
            c[i, i + s] = -2.0
        b = c.max(1)
        best.append(b.values)
        arg.append(b.indices)
    return torch.cat(best), torch.cat(arg)


def angle_to(v, j, rows):
    """Angle between unit rows and the unit vectors v[j], by half-chords (exact for small ones)."""
    return 2 * torch.asin((0.5 * (rows - v[j]).norm(dim=1)).clamp(max=1.0))


def spread(v):
    """Angle of each unit vector to the nearest other one."""
    return angle_to(v, nearest(v, v, skip_self=True)[1], v)


def genetic_children(x, slots, n, t, seed):
    """Random mating, SBX and polynomial mutation (distribution indices 20, box [0, 1])."""
    d, pairs, nv = x.shape[1], (n + 1) // 2, len(slots)
    w = philox(0, torch.arange(pairs, device=DEV), t, 1, seed)
    x1, x2 = (x[slots[(w[k] * nv) >> 32]] for k in (0, 1))
    w = gene_words(pairs, d, t, 2, seed)
    u = u24(w)
    beta = torch.where(u < 0.5, (2 * u) ** (1 / 21), (2 - 2 * u) ** (-1 / 21))
    beta = torch.where((w >> 7) & 1 == 1, beta, -beta)
    beta = torch.where((w >> 6) & 1 == 1, torch.ones_like(beta), beta)
    y = torch.cat([((1 + beta) * x1 + (1 - beta) * x2) / 2, ((1 - beta) * x1 + (1 + beta) * x2) / 2])
    y = y[:n].clamp(0.0, 1.0)
    w = philox(torch.arange(SITES, device=DEV)[None, :], torch.arange(n, device=DEV)[:, None], t, 4, seed)
    gap = torch.floor(torch.log(1.0 - u53(w[0], w[1])) / math.log1p(-1.0 / d))
    site = torch.cumsum(gap.clamp(max=d) + 1, 1).long() - 1
    child, e = torch.nonzero(site < d, as_tuple=True)
    site, u = site[child, e], u53(w[2], w[3])[child, e]
    g = y[child, site]
    low = (2 * u + (1 - 2 * u) * (1 - g) ** 21) ** (1 / 21) - 1
    high = 1 - (2 * (1 - u) + 2 * (u - 0.5) * g ** 21) ** (1 / 21)
    y[child, site] = (g + torch.where(u < 0.5, low, high)).clamp(0.0, 1.0)
    return y


def other_children(op, x, f, slots, n, t, seed):
    """Children of the other operators from a population at rest, default parameters."""
    d, nv, pairs = x.shape[1], len(slots), (n + 1) // 2
    units = pairs if op == "cso" else n
    who = torch.arange(units, device=DEV)
    pick = torch.stack([(k * nv) >> 32 for s in range(18) for k in philox(s, who, t, 5, seed)], 1)
    if op == "rand":
        return u24(gene_words(n, d, t, 6, seed))
    if op == "pso":
        xi, xl = x[slots[pick[:, 0]]], x[slots[pick[:, 1]]]
        return (xi + 1.5 * u24(gene_words(n, d, t, 6, seed)) * (xl - xi)).clamp(0.0, 1.0)
    if op == "cso":
        a, b = slots[pick[:, 0]], slots[pick[:, 1]]
        fa, fb = f[a].sum(1), f[b].sum(1)
        first = (fa < fb) | ((fa == fb) & (a <= b))
        win, lose = x[torch.where(first, a, b)], x[torch.where(first, b, a)]
        r2 = torch.stack([u24(philox(g, who, t, 6, seed)[1]) for g in range(d)], 1)
        return torch.cat([(lose + r2 * (win - lose)).clamp(0.0, 1.0), win])[:n]
    taken = [pick[:, 0]]  # DE: the target, then three donors
    forced = (philox(0, who, t, 5, seed)[1] * d) >> 32
    at = torch.full_like(who, 2)
    for _ in range(3):
        c = pick.gather(1, at[:, None])[:, 0]
        while nv >= 4:
            clash = torch.stack([c == o for o in taken]).any(0) & (at < 66)
            if not bool(clash.any()):
                break
            at = at + clash.long()
            c = pick.gather(1, at[:, None])[:, 0]
        taken.append(c)
        at = at + 1
    xt, a, b, c = (x[slots[k]] for k in taken)
    take = u24(gene_words(n, d, t, 6, seed)) < 0.9
    take[who, forced] = True
    return torch.where(take, (a + 0.5 * (b - c)).clamp(0.0, 1.0), xt)


def evolved(case, x, f, valid, seed):
    """The population after the case's generations, as get_state lays it out."""
    n, d, m, K = shape(case)
    v0 = simplex_vectors(m, K)
    v, gamma = v0, spread(v0)
    slots = torch.nonzero(valid)[:, 0]
    for t in range(1, case["gens"] + 1):
        if case["op"] == "ga":
            y = genetic_children(x, slots, n, t, seed)
        else:
            y = other_children(case["op"], x, f, slots, n, t, seed)
        y = y.float().double()  # genes are stored in 32 bits
        genes = torch.cat([x[slots], y])
        fm = torch.cat([f[slots], objectives(case["problem"], m, y)])
        fp = fm - fm.min(0).values
        norm = fp.norm(dim=1)
        unit = fp / norm.clamp(min=1e-300)[:, None]
        j = nearest(unit, v)[1]
        apd = (1 + m * (t / 100) ** 2 * angle_to(v, j, unit) / gamma[j]) * norm
        j = torch.where(norm > 0, j, torch.zeros_like(j))
        # least APD of each vector, the first row on ties: sort by APD, then (stably) by vector
        order = torch.argsort(torch.where(norm > 0, apd, 0 * apd), stable=True)
        order = order[torch.argsort(j[order], stable=True)]
        first = torch.ones_like(order, dtype=torch.bool)
        first[1:] = j[order][1:] != j[order][:-1]
        keep = order[first]
        slots = j[keep]
        x, f = torch.zeros(K, d, device=DEV, dtype=torch.float64), torch.full((K, m), math.nan, device=DEV, dtype=torch.float64)
        x[slots], f[slots] = genes[keep], fm[keep]
        if t % 10 == 0:
            v = v0 * (fm[keep].max(0).values - fm[keep].min(0).values)
            v = v / v.norm(dim=1, keepdim=True)
            gamma = spread(v)
    mask = torch.zeros(K, dtype=torch.uint8, device=DEV)
    mask[slots] = 1
    out = dict(X=x, F=f, valid=mask, V=v, V0=v0, gamma=gamma, t=case["gens"])
    out = {k: a.cpu().numpy() if torch.is_tensor(a) else a for k, a in out.items()}
    if case["kind"] == "evolve":
        out["X"] = None
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "indicators":
        return exact_indicators(case, seed)
    if kind in ("policy", "batch"):
        return None  # rounding to bfloat16 between the layers, or a long chain of choices, decides them
    n, d, m, K = shape(case)
    # Each selection chooses between neighbouring vectors; rounding the objectives to 32 bits tips
    # about one choice in 10^5, and one that is tipped changes every later generation.  So chains of
    # generations have a 64-bit value only where they are small, single generations always.
    if kind == "generation":
        x, f, valid = host_population(case, seed)
        x, f = torch.from_numpy(x).to(DEV).double(), torch.from_numpy(f).to(DEV).double()
        return evolved(case, x, f, torch.from_numpy(valid).to(DEV), seed)
    if case["op"] == "ga" and case["gens"] * (n + K) <= 25000 and n * d <= 10 ** 6:
        x = torch.zeros(K, d, device=DEV, dtype=torch.float64)
        x[:n] = u24(gene_words(n, d, 0, 0, seed))
        f = torch.full((K, m), math.nan, device=DEV, dtype=torch.float64)
        f[:n] = objectives(case["problem"], m, x[:n])
        valid = torch.zeros(K, dtype=torch.uint8, device=DEV)
        valid[:n] = 1
        return evolved(case, x, f, valid, seed)
    return dict(X=None, F=None, valid=None, V=None, V0=simplex_vectors(m, K).cpu().numpy(),
                gamma=None, t=None)


def exact_indicators(case, seed):
    f, valid = front(case, seed)
    f = f[valid == 1].double() / 1.1
    w = torch.from_numpy(weight_lattice(case["m"], case["weights"])).to(DEV)
    eu = float((-(w @ f.T)).max(1).values.mean())
    p = f[(f < 1).all(1)]
    z = p[:, 2] if case["m"] == 3 else torch.zeros(len(p), device=DEV, dtype=torch.float64)
    p, z = (a[torch.argsort(p[:, 0], stable=True)] for a in (p, z))
    width = torch.diff(p[:, 0], append=torch.ones(1, device=DEV, dtype=torch.float64))
    place = torch.empty(len(p), dtype=torch.long, device=DEV)
    place[torch.argsort(z, stable=True)] = torch.arange(len(p), device=DEV)
    hv = 0.0
    for s in range(0, len(p), 512):
        at = place[s:s + 512, None]
        y = torch.where(place[None, :] < at, p[None, :, 1], torch.ones((), device=DEV, dtype=torch.float64))
        low = torch.cummin(y, 1).values
        # the part of each rectangle that no earlier point covers
        right = torch.arange(len(p), device=DEV)[None, :] >= torch.arange(s, s + len(at), device=DEV)[:, None]
        area = ((low - p[s:s + 512, 1:2]).clamp(min=0) * width * right).sum(1)
        hv += float(((1 - z[s:s + 512]) * area).sum())
    return dict(hypervolume=hv, expected_utility=eu)
