"""The workloads whose speed is watched, through the public entry points.

A case is a dict of plain values.  ``listed()`` names the fixed ones,
``draw(rng)`` gives another of the same ranges, ``prepare`` builds what a
program has in hand before the call (graphs in device memory, right-hand
sides, score vectors, a batch handle), ``run`` is one pass, ``work`` the bytes
and operations a pass cannot do without and ``exact`` the same results from
plain torch in 64 bits.

Kinds:
  farness  forest farness, closeness and the diagonal of every vertex
  sample   trees with their per-tree outputs (parents, visits, digests)
  noalloc  the same trees from a loop that may not allocate device memory
  batch    many graphs at several alphas in one prepared launch
  solve    (alpha L + I) X = B for a block of right-hand sides
  group    the greedy vertex group of highest forest closeness
  rank     a ranking by score and Kendall's tau-b against another ranking
"""
import math

import numpy as np
import torch

import paper_2101_06192_amd as fc

DEV = "cuda:0"
MASK = 0xFFFFFFFF
RMAT = (0.57, 0.19, 0.19)


# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: a thousand vertices, tau from eps = delta = 0.1;
        # launches and host work count as much as the trees
        {"name": "farness_er1000", "kind": "farness", "graph": "er", "n": 1000, "deg": 5,
         "alpha": 1.0, "weighted": False, "tau": 0},
        # a serving loop that asks for a few trees of a small graph at a time
        {"name": "noalloc_er1000_64", "kind": "noalloc", "graph": "er", "n": 1000, "deg": 5,
         "alpha": 1.0, "weighted": False, "trees": 64},
        # the trees themselves (parents and visit counts of every vertex), for a
        # program that goes on with them
        {"name": "sample_ba20k_256", "kind": "sample", "graph": "ba", "n": 20000, "deg": 5,
         "alpha": 1.0, "weighted": False, "trees": 256},
        # a complex network of ordinary size, many trees (the benchmark's default)
        {"name": "farness_ba200k_4096", "kind": "farness", "graph": "ba", "n": 200000, "deg": 5,
         "alpha": 1.0, "weighted": False, "tau": 4096},
        # the same with edge weights, at the accuracy eps = delta = 0.1 asks for
        {"name": "farness_ba200k_w", "kind": "farness", "graph": "ba", "n": 200000, "deg": 5,
         "alpha": 1.0, "weighted": True, "tau": 0},
        # a road network: degree at most 4, neighbours close in id, disconnected
        {"name": "farness_grid1m", "kind": "farness", "graph": "grid", "n": 1000000, "deg": 2,
         "alpha": 1.0, "weighted": False, "tau": 1024},
        # the largest graph: heavy-tailed, four million vertices, eps = delta = 0.1
        {"name": "farness_rmat4m", "kind": "farness", "graph": "rmat", "n": 4194304, "deg": 8,
         "alpha": 1.0, "weighted": False, "tau": 0},
        # many graphs of uneven size at three alphas, prepared once and run
        {"name": "batch_rmat21x3_512", "kind": "batch", "graphs": 21, "lo_exp": 10.0,
         "hi_exp": 17.0, "deg": 8, "trees": 512, "autotune": True},
        # ground truth columns of a large network, 64 at a time
        {"name": "solve_ba2m_64_f32r", "kind": "solve", "graph": "ba", "n": 2000000, "deg": 8,
         "alpha": 1.0, "weighted": False, "rhs": 64, "precision": "fp32_refined", "rtol": 1e-9},
        # a few columns of an ordinary one, in binary64 throughout
        {"name": "solve_ba200k_8_f64", "kind": "solve", "graph": "ba", "n": 200000, "deg": 5,
         "alpha": 1.0, "weighted": False, "rhs": 8, "precision": "fp64", "rtol": 1e-10},
        # a vertex group in a graph of the size the group experiments use
        {"name": "group_ba2708_200", "kind": "group", "graph": "ba", "n": 2708, "deg": 2,
         "alpha": 1.0, "weighted": False, "k": 200},
        # the ranking of an estimate, and how well it agrees with the ground truth
        {"name": "rank_200k", "kind": "rank", "n": 200000, "tau": 841},
    ]


def _log(rng, lo, hi):
    """A whole number, its logarithm uniform in [log lo, log hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _network(rng, lo, hi):
    """A graph family with a size it is met in."""
    graph = rng.choice(["er", "ba", "ba", "rmat", "grid"])
    n = _log(rng, lo, min(hi, 400000) if graph == "er" else hi)
    deg = {"er": rng.choice([4, 5, 8]), "ba": rng.choice([2, 3, 5, 8]), "rmat": 8, "grid": 2}[graph]
    return {"graph": graph, "n": n, "deg": deg}


def draw(rng):
    kind = rng.choice(["farness"] * 5 + ["sample", "noalloc", "batch", "solve", "solve", "group", "rank"])
    if kind == "farness":
        c = _network(rng, 1000, 2000000)
        # trees: what eps = delta = 0.1 asks for, or a number of the caller's
        tau = rng.choice([0, _log(rng, 64, 4096)])
        c["alpha"] = rng.choice([0.5, 1.0, 1.0, 2.0])
        if c["n"] <= 100000 and rng.random() < 0.3:
            c["alpha"] = rng.choice([0.1, 10.0])
        return {"kind": kind, **c, "weighted": rng.random() < 0.25 and c["n"] <= 500000,
                "tau": min(tau, int(1.5e9 // c["n"]))}
    if kind in ("sample", "noalloc"):
        c = _network(rng, 500, 50000)
        return {"kind": kind, **c, "alpha": rng.choice([0.5, 1.0, 2.0]),
                "weighted": kind == "sample" and rng.random() < 0.25, "trees": _log(rng, 16, 512)}
    if kind == "batch":
        lo = rng.uniform(9.0, 12.0)
        return {"kind": kind, "graphs": rng.randint(3, 21), "lo_exp": lo,
                "hi_exp": lo + rng.uniform(1.0, 5.0), "deg": 8, "trees": _log(rng, 32, 512),
                "autotune": rng.random() < 0.5}
    if kind == "solve":
        c = _network(rng, 5000, 1000000)
        return {"kind": kind, **c, "alpha": rng.choice([0.5, 1.0, 2.0]),
                "weighted": rng.random() < 0.25, "rhs": rng.choice([1, 3, 8, 17, 32, 64]),
                "precision": rng.choice(["fp64", "fp32_refined"]), "rtol": rng.choice([1e-9, 1e-10])}
    if kind == "group":
        n = _log(rng, 500, 5000)
        return {"kind": kind, "graph": rng.choice(["ba", "er"]), "n": n, "deg": rng.choice([2, 3]),
                "alpha": rng.choice([0.5, 1.0]), "weighted": rng.random() < 0.25,
                "k": _log(rng, 5, min(300, n // 4))}
    return {"kind": kind, "n": _log(rng, 1000, 2000000), "tau": _log(rng, 81, 2000)}


# --------------------------------------------------------------------------
# Inputs, made on the GPU from the seed alone
# --------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _edges(case, gen):
    """The endpoints of the edges, by the graph family's recipe (int64; loops and
    repeats are dropped later)."""
    n, deg = case["n"], case["deg"]

    def ints(hi, count):
        return torch.randint(hi, (count,), generator=gen, device=DEV)

    if case["graph"] == "grid":  # rows in id order, 12% of the edges removed
        cols = max(2, int(math.isqrt(n)))
        v = torch.arange(n, device=DEV)
        right, down = v[(v % cols != cols - 1) & (v + 1 < n)], v[v + cols < n]
        u, w = torch.cat([right, down]), torch.cat([right + 1, down + cols])
        keep = torch.rand(u.numel(), generator=gen, device=DEV) >= 0.12
        return u[keep], w[keep]
    if case["graph"] == "er":
        return ints(n, n * deg), ints(n, n * deg)
    if case["graph"] == "ba":
        # each vertex attaches to `deg` earlier ones picked from the list of edge
        # endpoints: a pick of another edge's target is followed to its source
        m = deg
        clique = torch.triu_indices(m + 1, m + 1, 1, device=DEV)
        e0 = clique.shape[1]
        src = torch.cat([clique[0], torch.arange(m + 1, n, device=DEV).repeat_interleave(m)])
        first = e0 + (torch.arange(src.numel() - e0, device=DEV) // m) * m
        pick = (torch.rand(first.numel(), generator=gen, device=DEV, dtype=torch.float64) * (2 * first)).long()
        at = pick.clone()
        while True:
            more = (at % 2 == 1) & (at >= 2 * e0)
            if not bool(more.any()):
                break
            at = torch.where(more, pick[(at // 2 - e0).clamp_(min=0)], at)
        known = torch.where(at % 2 == 0, src[at // 2], clique[1][(at // 2).clamp(max=e0 - 1)])
        u, v = src, torch.cat([clique[1], known])
    else:  # rmat: quadrant by quadrant, draws outside [0, n) drawn again
        scale, want = max(1, math.ceil(math.log2(n))), deg * n
        us, vs, have = [], [], 0
        a, b, c = RMAT
        while have < want:
            count = want - have + 1024 if have else want
            u = torch.zeros(count, dtype=torch.int64, device=DEV)
            v = torch.zeros_like(u)
            for _ in range(scale):
                r = torch.rand(count, generator=gen, device=DEV)
                u = 2 * u + (r >= a + b)
                v = 2 * v + (((r >= a) & (r < a + b)) | (r >= a + b + c))
            ok = (u < n) & (v < n)
            us.append(u[ok])
            vs.append(v[ok])
            have += us[-1].numel()
        u, v = torch.cat(us)[:want], torch.cat(vs)[:want]
    new = torch.randperm(n, generator=gen, device=DEV)
    return new[u], new[v]


def _graph(case, seed):
    """The case's graph in device memory: simple, symmetric, rows ascending."""
    gen = _generator(seed)
    n = case["n"]
    u, v = _edges(case, gen)
    keep = u != v
    u, v = u[keep], v[keep]
    und = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    lo, hi = und // n, und % n
    key, order = torch.sort(torch.cat([und, hi * n + lo]))
    row_ptr = torch.searchsorted(key, torch.arange(n + 1, device=DEV) * n).int()
    weights = None
    if case["weighted"]:  # log-uniform in [0.1, 10), the same in both directions
        w = 0.1 * torch.pow(100.0, torch.rand(und.numel(), generator=gen, device=DEV, dtype=torch.float64))
        weights = torch.cat([w, w])[order].contiguous()
    return fc.DeviceGraph(n, row_ptr.contiguous(), (key % n).int().contiguous(), weights)


def _batch_cases(case):
    """Sizes spread evenly over [lo_exp, hi_exp] in the logarithm."""
    q, span = case["graphs"], case["hi_exp"] - case["lo_exp"]
    return [{"graph": "rmat", "deg": case["deg"], "weighted": False,
             "n": int(round(2.0 ** (case["lo_exp"] + span * (i + 0.5) / q)))} for i in range(q)]


ALPHAS = (0.1, 1.0, 10.0)


def _scores(case, seed):
    """A diagonal of the forest matrix as degrees shape it, and its estimate from
    tau trees: whole multiples of 1 / tau, so with many ties."""
    gen = _generator(seed)
    n, tau = case["n"], case["tau"]
    degree = 5.0 / torch.rand(n, generator=gen, device=DEV, dtype=torch.float64).clamp_(min=1e-6).sqrt()
    noise = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
    truth = (1.0 + 0.1 * noise).clamp_(0.5, 1.5) / (1.0 + degree)
    sd = (tau * truth * (1.0 - truth)).sqrt()
    est = (tau * truth + sd * torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)).round()
    return truth, est.clamp_(0, tau) / tau


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case, "seed": int(seed)}
    if kind == "rank":
        state["truth"], state["est"] = _scores(case, seed)
    elif kind == "batch":
        graphs = [_graph(c, seed * 1009 + i) for i, c in enumerate(_batch_cases(case))]
        jobs = [{"graph": g, "alpha": a, "tree_count": case["trees"], "stream_id": i}
                for i, g in enumerate(graphs) for a in ALPHAS]
        state["batch"] = fc.Batch(jobs, seed=seed, autotune=case["autotune"])
    else:
        state["graph"] = _graph(case, seed)
        if kind == "solve":
            state["B"] = torch.randn(case["n"], case["rhs"], generator=_generator(seed + 1), device=DEV,
                                     dtype=torch.float64)
    return state


def run(state):
    c, g, seed = state["case"], state.get("graph"), state["seed"]
    kind = c["kind"]
    if kind == "farness":
        r = fc.farness(g, alpha=c["alpha"], eps=0.1, delta=0.1, tau=c["tau"], seed=seed, as_torch=True)
        return {"farness": r["farness"], "closeness": r["closeness"], "diag": r["diag"],
                "root_counts": r["root_counts"], "tau": r["tau"], "steps": r["stats"]["walk_steps"]}
    if kind == "sample":
        r = fc.sample(g, c["alpha"], seed=seed, tree_count=c["trees"], as_torch=True, want_visits=True,
                      want_digests=True, want_steps=True, want_parents=True, want_tree_visits=True)
        return {k: v for k, v in r.items() if k != "stats"}
    if kind == "noalloc":
        r = fc.sample_noalloc(g, c["alpha"], seed=seed, tree_count=c["trees"], as_torch=True,
                              want_digests=True)
        return {k: v for k, v in r.items() if k != "stats"}
    if kind == "batch":
        b = state["batch"]
        b.reset()
        b.run()
        return {"root_counts": b.root_counts}
    if kind == "solve":
        return {"X": fc.solve(g, c["alpha"], state["B"], rtol=c["rtol"], precision=c["precision"],
                              as_torch=True)["X"]}
    if kind == "group":
        r = fc.group_closeness(g, c["alpha"], c["k"])
        return {"group": np.array(r["group"]), "farness": np.array(r["farness"])}
    order = fc.rank(state["est"], as_torch=True)
    kt = fc.kendall_tau(state["est"], state["truth"])
    return {"order": order["order"], "rank": order["rank"], "tau_b": kt["tau_b"], "counts": np.array(kt["counts"])}


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

def _trees(case):
    t = case.get("trees", case.get("tau", 0))
    return t if t else fc.tau(case["n"] * case["deg"], case["n"], 0.1, 0.1)


def work(case):
    kind, n = case["kind"], case.get("n", 0)
    arrow = 70.0  # operations of one Philox4x32-10 block and its step
    if kind == "rank":
        # both vectors read, order and rank written; a comparison per level and element
        return {"bytes": 16.0 * n + 8.0 * n, "flops": 2.0 * n * math.log2(max(2, n))}
    if kind == "batch":
        sizes = [c["n"] for c in _batch_cases(case)]
        return {"bytes": sum((4 + 8 * case["deg"] + 4 * len(ALPHAS)) * s for s in sizes),
                "flops": arrow * len(ALPHAS) * case["trees"] * sum(sizes)}
    csr = 4.0 * n + 8.0 * n * case["deg"] * (3 if case["weighted"] else 1)
    if kind == "solve":
        # the operator about twenty times, right-hand sides in, solutions out
        return {"bytes": csr + 16.0 * n * case["rhs"],
                "flops": 20.0 * case["rhs"] * (4.0 * n * case["deg"] + 10.0 * n)}
    if kind == "group":
        return {"bytes": csr + 8.0 * n * n, "flops": 2.0 * n ** 3 + 4.0 * n * n * case["k"]}
    trees = _trees(case)
    out = 28.0 * n if kind == "farness" else 4.0 * n + 8.0 * trees
    if kind == "sample":
        out += 8.0 * n + 8.0 * trees + 8.0 * n * trees
    return {"bytes": csr + out, "flops": arrow * n * trees}


# --------------------------------------------------------------------------
# The same results from plain torch
# --------------------------------------------------------------------------

def _philox(c, key):
    """Philox4x32-10 (Salmon et al., SC 2011) on int64 tensors of 32-bit words:
    the first two output words."""
    c0, c1, c2, c3 = c
    k0, k1 = key
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wraps: the high word is masked below
        c0, c1, c2, c3 = (((p1 >> 32) & MASK) ^ c1 ^ k0, p1 & MASK, ((p0 >> 32) & MASK) ^ c3 ^ k1, p0 & MASK)
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1


def _root_counts(g, alpha, seed, trees):
    """How often each vertex hangs off the universal vertex in `trees` uniform
    spanning trees: cycle popping, all cycles of all trees at once."""
    n = g.n
    rp, col = g.row_ptr.long(), g.col_idx.long()
    d = rp[1:] - rp[:-1]
    if g.weights is None:
        w = d.double()
    else:
        run_ = torch.cat([torch.zeros(1, device=DEV, dtype=torch.float64), g.weights.cumsum(0)])
        w = run_[rp[1:]] - run_[rp[:-1]]
    thr = torch.floor(4294967296.0 * (1.0 / (alpha * w + 1.0))).long()
    thr[d == 0] = 1 << 32
    key = (seed & MASK, (seed >> 32) & MASK)
    counts = torch.zeros(n, dtype=torch.int64, device=DEV)
    hops = max(1, math.ceil(math.log2(n + 1)))
    chunk = max(1, int(3e7 // (n + 1)))
    for t0 in range(0, trees, chunk):
        tc = min(chunk, trees - t0)
        flat = torch.arange(tc * (n + 1), device=DEV)
        vert = flat[flat % (n + 1) != n]  # the last place of a tree is the root, its own successor

        def arrows(at, j):
            t, v = at // (n + 1), at % (n + 1)
            x0, x1 = _philox((v, j, t + t0, torch.zeros_like(v)), key)
            if g.weights is None:
                e = rp[v] + ((x1 * d[v]) >> 32)
            else:
                e = torch.searchsorted(run_, run_[rp[v]] + x1.double() * w[v] * 2.0 ** -32, right=True) - 1
                e = torch.minimum(torch.maximum(e, rp[v]), rp[v + 1] - 1)
            to = col[e.clamp(max=max(0, col.numel() - 1))] if col.numel() else torch.zeros_like(v)
            return torch.where(x0 < thr[v], n, to) + t * (n + 1)

        nxt = flat.clone()
        draws = torch.zeros_like(flat)
        nxt[vert] = arrows(vert, torch.zeros_like(vert))
        jump, open_ = nxt.clone(), vert
        while open_.numel():
            for _ in range(hops):  # 2^hops steps: at the root, or on a cycle
                jump[open_] = jump[jump[open_]]
            far = jump[open_]
            left = far % (n + 1) != n
            open_ = open_[left]
            if not open_.numel():
                break
            cycle = torch.unique(far[left])
            draws[cycle] += 1
            nxt[cycle] = arrows(cycle, draws[cycle])
            jump[open_] = nxt[open_]
        rooted = vert[nxt[vert] % (n + 1) == n] % (n + 1)
        counts += torch.bincount(rooted, minlength=n)
    return counts


def _solution(g, alpha, B):
    """Jacobi-preconditioned conjugate gradients in binary64, to the last digits."""
    n = g.n
    w = g.weights if g.weights is not None else torch.ones(g.nnz, device=DEV, dtype=torch.float64)
    adj = torch.sparse_csr_tensor(g.row_ptr, g.col_idx, w, size=(n, n))
    diag = 1.0 + alpha * (adj @ torch.ones(n, 1, device=DEV, dtype=torch.float64))
    X = torch.zeros_like(B)
    R = B.clone()
    P = Z = R / diag
    rz, b2 = (R * Z).sum(0), (B * B).sum(0)
    for _ in range(400):
        Q = diag * P - alpha * (adj @ P)
        a = rz / (P * Q).sum(0).clamp(min=1e-300)
        X, R = X + a * P, R - a * Q
        if bool(((R * R).sum(0) <= 1e-28 * b2).all()):
            break
        Z = R / diag
        rz, old = (R * Z).sum(0), rz
        P = Z + rz / old.clamp(min=1e-300) * P
    return X


def _group_farness(g, alpha, k):
    """The greedy group's trace after each choice, on dense matrices."""
    n = g.n
    deg = (g.row_ptr[1:] - g.row_ptr[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    w = g.weights if g.weights is not None else torch.ones(g.nnz, device=DEV, dtype=torch.float64)
    A = torch.zeros(n, n, device=DEV, dtype=torch.float64)
    A[rows, g.col_idx.long()] = -alpha * w
    A.diagonal().copy_(1.0 - A.sum(1))
    om = torch.linalg.inv(A)
    first = int(om.diagonal().argmin())
    # grounded at the first vertex, the universal vertex in its place
    c, c0 = om[:, first].clone(), om[first, first].clone()
    om[first, :] = 0.0
    om[:, first] = 0.0
    c[first] = 0.0
    M = om - c[:, None] - c[None, :] + c0
    taken = torch.zeros(n, dtype=torch.bool, device=DEV)
    taken[first] = True
    out = [M.trace()]
    for _ in range(k - 1):
        gain = (M * M).sum(0) / M.diagonal()
        v = int(torch.where(taken, -math.inf, gain).argmax())
        taken[v] = True
        m, d = M[:, v].clone(), M[v, v].clone()
        M -= torch.outer(m, m / d)
        M[v, :] = 0.0
        M[:, v] = 0.0
        out.append(M.trace())
    return torch.stack(out)


def _tau_b(a, b):
    """Kendall's tau-b from its pair counts."""
    n = a.numel()
    ra, rb = (torch.unique(x, return_inverse=True)[1] for x in (a, b))

    def tied(x):
        q = torch.unique(x, return_counts=True)[1]
        return int((q * (q - 1) // 2).sum())

    n0, na, nb, nab = n * (n - 1) // 2, tied(ra), tied(rb), tied(ra * n + rb)
    seq = rb[torch.argsort(ra * n + rb, stable=True)]
    bits = max(1, int(seq.max()).bit_length())
    nd, group = 0, torch.zeros(n, dtype=torch.int64, device=DEV)
    for bit in range(bits - 1, -1, -1):  # within equal higher bits: ones that stand before zeros
        one = (seq >> bit) & 1
        before = one.cumsum(0) - one
        start = torch.searchsorted(group, group)
        nd += int(((before - before[start]) * (1 - one)).sum())
        group = 2 * group + one
        group, order = torch.sort(group, stable=True)
        seq = seq[order]
    nc = n0 - na - nb + nab - nd
    return (nc - nd) / math.sqrt(float((n0 - na)) * float((n0 - nb)))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sample", "noalloc", "batch"):
        return None  # whole numbers only
    if kind == "rank":
        truth, est = _scores(case, seed)
        return {"order": None, "rank": None, "tau_b": _tau_b(est, truth), "counts": None}
    if kind == "farness" and case["n"] * _trees(case) > 1.2e9:
        return None  # too long
    g = _graph(case, seed)
    if kind == "group":
        return {"group": None, "farness": _group_farness(g, case["alpha"], case["k"]).cpu().numpy()}
    if kind == "solve":
        B = torch.randn(case["n"], case["rhs"], generator=_generator(seed + 1), device=DEV, dtype=torch.float64)
        return {"X": _solution(g, case["alpha"], B)}
    # the sample size of Algorithm 1 at eps = delta = 0.1
    tau = case["tau"] if case["tau"] else math.ceil(math.log(2.0 * max(g.m, g.n) / 0.1) / 0.02)
    counts = _root_counts(g, case["alpha"], seed, tau).double()
    farness = (g.n * counts + counts.sum()) / tau - 2.0
    return {"farness": farness, "closeness": g.n / farness, "diag": counts / tau, "root_counts": None,
            "tau": None, "steps": None}
