"""Timed work of the library: what its users have it do, through the public
entry points of paper_2605_09950_amd.binding.

listed() holds the workloads of bench.py and of the tests by shape (seeded
random inputs of the same recipes), from a small problem whose time is launches
and host calls to the 100,000 x 2,000 matrix past the last-level cache, in the
three importance modes and for both kinds of forest; draw() gives others of
the same ranges.  prepare() makes a case's inputs (and the workspace that a
program keeps), run() is one whole call: set-up with binning, the iterations
and the read-back of every result.

Every result is a deterministic function of the inputs: hits and decisions are
integers, and each reported importance is one float64 quotient of exact
integers, so runs compare bit for bit.
"""
import math

import numpy as np
import torch

from paper_2605_09950_amd import binding as B

MODES = {"treeimp": B.TREEIMP, "permut": B.PERMUT, "divergence": B.PERMUT_KL}


def _case(entry, data, n, p, k, trees, depth, iters, mode="treeimp", bins=256, n_perm=1,
          jobs=1, rank="fp32", mtry=0, name=None):
    c = dict(entry=entry, data=data, n=n, p=p, classes=k, trees=trees, depth=depth, iters=iters,
             mode=mode, bins=bins, n_perm=n_perm, jobs=jobs, rank=rank, mtry=mtry)
    if name:
        c["name"] = name
    return c


def listed():
    """classes = 0: a regression forest."""
    return [
        # a quick look at a small table from host arrays: launches and host
        # calls are the cost (the planted recovery check's shape)
        _case("fit", "planted", 500, 20, 2, 50, 8, 20, bins=64, name="planted_fit"),
        # a caller that may not allocate (a serving loop): the largest problem
        # of the tests that the library's own scratch takes, launched eagerly
        _case("noalloc", "planted", 3000, 120, 3, 60, 10, 12, mode="permut",
              name="noalloc_permut"),
        # the paper's MADELON shape, run until every feature is decided, on
        # device-resident inputs with a workspace: TreeImp
        _case("device", "madelon", 10000, 500, 3, 200, 12, 100, name="madelon_treeimp"),
        # the same by out-of-bag accuracy drop, the first iterations
        _case("device", "madelon", 10000, 500, 3, 200, 12, 20, mode="permut",
              name="madelon_permut"),
        # the same by prediction divergence (Algorithm 3)
        _case("device", "madelon", 10000, 500, 3, 200, 12, 8, mode="divergence",
              name="madelon_divergence"),
        # omics tables: few rows, very many columns, two classes
        _case("device", "omics", 2000, 20000, 2, 500, 12, 12, name="omics_treeimp"),
        # many independent jobs of mixed shapes and class counts (n and p are
        # the largest job's) advanced together in one session
        _case("session", "jobs", 5000, 2000, 5, 100, 10, 6, mode="permut", jobs=64,
              name="many_jobs_permut"),
        # more classes than four, ragged sizes, exact-only split ranking (the
        # option that trusts no floating-point ranking)
        _case("fit", "planted", 5003, 257, 7, 100, 13, 8, rank="exact", name="classes7_exact"),
        # the largest matrix: mixed types, past the last-level cache; the
        # first iterations, when every column is still in the race
        _case("device", "mixed", 100000, 2000, 4, 300, 16, 4, name="mixed_treeimp"),
        # the same by accuracy drop with five replicas
        _case("device", "mixed", 100000, 2000, 4, 300, 16, 2, mode="permut", n_perm=5,
              name="mixed_permut"),
        # the paper's synthetic regression shape by TreeImp: a whole run where
        # every feature is decided early, else its first 40 iterations
        _case("session", "regression", 10000, 50, 0, 200, 12, 40, name="regression_treeimp"),
        # the repeated-seed protocol of the experiments on it, by squared-error
        # increase, from host arrays
        _case("seeds", "regression", 10000, 50, 0, 200, 12, 8, mode="permut", jobs=5,
              name="regression_seeds"),
    ]


def _depth_used(c):
    """Tree levels that hold rows to search (deeper ones are empty)."""
    return min(c["depth"], max(1, int(math.log2(max(2, c["n"])))))


def _mtry(c):
    return c["mtry"] or max(1, math.isqrt(2 * c["p"]))


def _rows(c):
    """Rows of all jobs of the case ("jobs": sizes spread down from n)."""
    if c["data"] == "jobs":
        return sum(n for n, _, _ in _job_shapes(c))
    return c["n"] * c["jobs"]


def _pairs(c):
    """(row, drawn column) pairs of one iteration's trees: each tree holds
    1 - 1/e of the rows at every level."""
    if c["data"] == "jobs":
        s = sum(n * math.isqrt(2 * p) for n, p, _ in _job_shapes(c))
    else:
        s = _rows(c) * _mtry(c)
    return 0.632 * s * c["trees"] * _depth_used(c)


def _cost(c):
    """Rough time of a case, to keep drawn ones within the listed range: row
    work, nodes, launches, the matrix, and the importance modes' routing."""
    it = min(c["iters"], 40)
    route = 0.632 * _rows(c) * c["trees"] * _depth_used(c)
    planes = 3 if c["data"] == "jobs" else 1 if c["classes"] <= 4 else 2.5 if c["classes"] <= 8 else 5
    per_it = planes * _pairs(c) / 3e11 + 60e-6 * c["depth"]
    if c["mode"] != "treeimp":
        per_it += route * _depth_used(c) * c["n_perm"] * (2 if c["mode"] == "divergence" else 1) / 6e10
    if c["mode"] == "divergence":
        per_it += 3e-12 * _rows(c) * c["p"] * max(c["classes"], 2)
    if c["classes"] == 0 or c["rank"] == "exact":
        per_it *= 2
    return it * per_it + 4e-10 * c["n"] * c["p"] + 5e-3


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["planted", "planted", "madelon", "omics", "mixed", "regression",
                           "jobs"])
        entry = {"planted": rng.choice(["fit", "device", "noalloc"]), "madelon": "device",
                 "omics": "device", "mixed": "device", "jobs": "session",
                 "regression": rng.choice(["session", "seeds"])}[kind]
        n, p = {"planted": (log(200, 6000), log(10, 400)),
                "madelon": (log(1000, 30000), log(100, 1200)),
                "omics": (log(150, 4000), log(3000, 20000)),
                "mixed": (log(8000, 100000), log(100, 2000)),
                "regression": (log(500, 20000), log(10, 300)),
                "jobs": (log(400, 5000), log(60, 2000))}[kind]
        if entry == "noalloc":
            n, p = min(n, 3000), min(p, 120)
        k = 0 if kind == "regression" else (5 if kind == "jobs" else
                                            rng.choice([2, 2, 3, 3, 4, 4, 6, 9, 16]))
        c = _case(entry, kind, n, p, k,
                  trees=log(20, 60) if entry == "noalloc" else log(30, 500),
                  depth=rng.randint(4, 10) if entry == "noalloc" else rng.randint(5, 16),
                  iters=rng.randint(2, 40), mode=rng.choice(list(MODES)[:2] * 2 + list(MODES)[2:]),
                  bins=rng.choice([256, 256, 256, 100, 64, 33]),
                  n_perm=1, jobs={"jobs": rng.randint(8, 64), "regression": 1}.get(kind, 1),
                  rank="exact" if rng.random() < 0.1 else "fp32",
                  mtry=rng.choice([0, 0, 0, max(1, p // 3)]) if kind == "planted" else 0)
        if entry == "seeds":
            c["jobs"] = rng.randint(2, 6)
        if c["mode"] == "permut":
            c["n_perm"] = rng.choice([1, 1, 3, 5])
        if kind == "jobs":
            c["trees"] = min(c["trees"], 100)
        while c["iters"] > 1 and _cost(c) > 0.2:
            c["iters"] = (c["iters"] + 1) // 2
        if _cost(c) <= 0.25:
            return c


def _job_shapes(c):
    """Shapes (n, p, classes) of a batch's jobs: spread evenly over their
    ranges, in an order that mixes them."""
    out = []
    for j in range(c["jobs"]):
        u = ((j * 37) % c["jobs"] + 0.5) / c["jobs"]
        v = ((j * 23 + 11) % c["jobs"] + 0.5) / c["jobs"]
        n = int(c["n"] * (0.04 + 0.96 * u))
        p = max(5, int(c["p"] * (0.025 + 0.975 * v)))
        out.append((max(50, n), p, 2 + j % (c["classes"] - 1)))
    return out


def _informative(p, k, gen):
    return torch.randperm(p, generator=gen, device="cuda")[:min(p, k)]


def _linear_label(X, inf, k, gen, noise=0.5):
    W = torch.randn(len(inf), k, generator=gen, device="cuda")
    s = X[:, inf] @ W + noise * torch.randn(len(X), k, generator=gen, device="cuda")
    return torch.argmax(s, dim=1).to(torch.int32)


def _problem(data, n, p, k, gen):
    """(X float32 [n][p], y) on the device, by the recipes of the synthetic
    workloads: Gaussian columns with a few that decide the label; noisy mixes
    of them; log-normal columns; mixed column types with a tree-shaped label;
    uniform columns with a smooth target."""
    dev = dict(generator=gen, device="cuda")
    if data in ("planted", "jobs"):
        X = torch.randn(n, p, **dev)
        return X, _linear_label(X, _informative(p, max(5, p // 20), gen), k, gen)
    if data == "madelon":
        n_inf, n_mix = max(2, p // 25), (p * 4) // 25
        XI = torch.randn(n, n_inf, **dev)
        s = torch.stack([((XI @ torch.randn(n_inf, n_inf, **dev)) * XI).sum(1)
                         for _ in range(k)], 1)
        mixes = XI @ torch.randn(n_inf, n_mix, **dev) / math.sqrt(n_inf)
        mixes = mixes + 0.1 * torch.randn(n, n_mix, **dev)
        X = torch.cat([XI, mixes, torch.randn(n, p - n_inf - n_mix, **dev)], 1)
        X = X[:, torch.randperm(p, **dev)].contiguous()
        return X, torch.argmax(s, dim=1).to(torch.int32)
    if data == "omics":
        Z = torch.randn(n, p, **dev)
        y = _linear_label(Z, _informative(p, 50, gen), k, gen)
        flip = torch.rand(n, **dev) < 0.1
        y = torch.where(flip, (y + 1) % k, y)
        return Z.exp_(), y
    if data == "mixed":
        X = torch.empty(n, p, device="cuda")
        kinds = torch.randperm(p, **dev)
        a, b = int(0.45 * p), int(0.9 * p)
        X[:, kinds[:a]] = torch.randn(n, a, **dev)
        X[:, kinds[a:b]] = torch.rand(n, b - a, **dev)
        levels = torch.randint(2, 17, (p - b,), **dev)
        X[:, kinds[b:]] = torch.floor(torch.rand(n, p - b, **dev) * levels)
        inf = _informative(p, 40, gen)
        depth = 6
        feat = inf[torch.randint(0, len(inf), (2 ** depth - 1,), **dev)]
        q = 0.2 + 0.6 * torch.rand(2 ** depth - 1, **dev)
        lo, hi = X[:, feat].amin(0), X[:, feat].amax(0)
        thr = torch.where(torch.rand(2 ** depth - 1, **dev) < 0.5, X[:, feat].median(0).values,
                          lo + q * (hi - lo))
        leaf = torch.randint(0, k, (2 ** depth,), **dev)
        node = torch.zeros(n, dtype=torch.int64, device="cuda")
        rows = torch.arange(n, device="cuda")
        for _ in range(depth):
            node = 2 * node + 1 + (X[rows, feat[node]] > thr[node]).long()
        return X, leaf[node - (2 ** depth - 1)].to(torch.int32)
    X = torch.rand(n, p, **dev)
    Z = X[:, _informative(p, 10, gen)]
    y = 5 * Z[:, 0] + 3 * torch.sin(math.pi * Z[:, 1] * Z[:, 2]) + 4 * (Z[:, 3] - 0.5) ** 2
    y = y + 2 * (Z[:, 4] > 0.5) + 1.5 * Z[:, 5] * Z[:, 6] + Z[:, 7] - Z[:, 8]
    y = y + 0.5 * torch.cos(2 * math.pi * Z[:, 9]) + 0.5 * torch.randn(n, **dev)
    return X, y.float()


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * seed + 17)
    shapes = _job_shapes(c) if c["data"] == "jobs" else [(c["n"], c["p"], c["classes"])]
    probs = [_problem(c["data"], n, p, k, gen) + (k,) for n, p, k in shapes]
    state = dict(case=c, seed=7000 + seed,
                 common=dict(max_iter=c["iters"], importance_mode=MODES[c["mode"]],
                             mtry=c["mtry"]),
                 options=dict(n_bins=c["bins"], n_perm=c["n_perm"],
                              split_rank=B.RANK_EXACT if c["rank"] == "exact" else B.RANK_FP32))
    if c["entry"] in ("fit", "seeds"):  # the call takes host arrays
        X, y, _ = probs[0]
        state["X"], state["y"] = X.cpu().numpy(), y.cpu().numpy()
        return state
    state["probs"] = probs
    if c["entry"] != "noalloc":
        sizes = [dict(n=X.shape[0], p=X.shape[1], n_classes=k or 2, n_trees=c["trees"],
                      max_depth=c["depth"], regression=k == 0, **state["common"])
                 for X, _, k in probs]
        nbytes = B.boruta_workspace_size(sizes, **state["options"])
        state["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    return state


def _whole(r):
    # rows past the last iteration and features rejected earlier hold NaN: -1 here
    return {"decision": r["decision"], "hits": r["hits"], "n_iter": r["n_iter"],
            "importance": np.nan_to_num(r["imp_history"], nan=-1.0),
            "shadow_max": np.nan_to_num(r["shadow_max"], nan=-1.0)}


def run(state):
    c, kw, opt = state["case"], state["common"], state["options"]
    T, D, seed = c["trees"], c["depth"], state["seed"]
    if c["entry"] == "fit":
        return _whole(B.boruta_fit_ex(state["X"], state["y"], c["classes"], T, D, seed=seed,
                                      **kw, **opt))
    if c["entry"] == "seeds":
        r = B.boruta_fit_seeds(state["X"], state["y"], c["classes"] or None, T, D,
                               [seed + 31 * s for s in range(c["jobs"])], **kw, **opt)
        return {"median": r["median_importance"], "decision": r["decision"],
                "runs": [_whole(s) for s in r["runs"]]}
    if c["entry"] in ("device", "noalloc"):
        X, y, k = state["probs"][0]
        if c["entry"] == "device":
            return _whole(B.boruta_fit_device(X, y, k, T, D, state["workspace"], seed=seed, **kw,
                                              **opt))
        return _whole(B.boruta_fit_device_noalloc(X, y, k, T, D, seed=seed, **kw, **opt))
    jobs = [dict({"y": y, "n_classes": k} if k else {"y_reg": y}, X=X, n_trees=T, max_depth=D,
                 seed=seed + j, **kw) for j, (X, y, k) in enumerate(state["probs"])]
    with B.Session(jobs, inputs_on_device=True, workspace=state["workspace"],
                   stream=torch.cuda.current_stream(), **opt) as s:
        s.run(c["iters"])
        rs = [s.result(j) for j in range(len(jobs))]
    if len(rs) <= 8:
        return [dict(_whole(r), rank=r["rank"]) for r in rs]
    # many jobs: each kind of result of all jobs in one array
    ws = [dict(_whole(r), rank=r["rank"]) for r in rs]
    return {key: np.concatenate([np.ravel(w[key]) for w in ws]) for key in ws[0]}


def work(case):
    """Bytes: the inputs, and for each iteration with every column still in the
    race (none can be rejected before 2^-t p < alpha) one bin byte per row of
    a node and drawn column, plus six bytes of row record per row and level.
    Operations: one addition per such pair."""
    full = min(case["iters"], max(1, math.ceil(math.log2(case["p"] / 0.05))))
    if case["entry"] == "seeds":
        matrix = case["n"] * case["p"]
    elif case["data"] == "jobs":
        matrix = sum(n * p for n, p, _ in _job_shapes(case))
    else:
        matrix = case["n"] * case["p"]
    rows = 0.632 * _rows(case) * case["trees"] * _depth_used(case)
    pairs = _pairs(case)
    return {"bytes": 4.0 * matrix + full * (pairs + 6.0 * rows), "flops": full * pairs}


def exact(case, seed):
    """None: a forest's numbers are integers at every step (and float64
    quotients of them at the end), defined by keyed draws; without the
    library's code a run is far past 20 seconds in numpy."""
    return None
