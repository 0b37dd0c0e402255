"""Performance cases of the framework: the calls a user makes, over the range they are made in.

Data come from linear vector-autoregressive processes and coupled logistic maps, the two kinds of
process the framework's searches are run on, or (single estimates) from jointly Gaussian samples.
Every case goes through a public entry point:

* ``estimate``   one KSG estimate on device tensors (cmi_ksg_dev)
* ``test``       one transfer-entropy test on device tensors: the estimate and its S permutation
                 surrogates (cmi_ksg_surrogates_dev)
* ``hosttest``   the same test from host arrays, also with replications (cmi_ksg_surrogates,
                 cmi_ksg_surrogates_rep)
* ``served``     a burst of unrelated tests through the request loop (mte_submit, mte_wait)
* ``network``    network inference over all targets (mte_infer_network)
* ``search``     the greedy source selection of one target (mte_select_sources)
* ``gauss``      the Gaussian estimator: a covariance matrix on the device and, when the case asks
                 for them, the estimates of a greedy round against it
"""

import math

import numpy as np
import torch

import paper_1902_06828_amd as mte

MAX_LAG = 5


def listed():
    return [
        # the smallest call: one estimate of a Gaussian triple, dominated by launches
        {"name": "estimate n1000 dz1", "kind": "estimate", "n": 1000, "dx": 1, "dz": 1, "k": 4, "theiler": 0},
        # one estimate per call at the usual series length (a caller without surrogates)
        {"name": "estimate n10000 dz5", "kind": "estimate", "n": 10000, "dx": 1, "dz": 5, "k": 4, "theiler": 0},
        # a short recording tested from host arrays, an odd number of rows
        {"name": "hosttest n1003 dz3", "kind": "hosttest", "n": 1003, "dx": 1, "dz": 3, "k": 4, "S": 200, "reps": 1},
        # the usual test: a source's past given five lags of the target
        {"name": "test n10000 dz5", "kind": "test", "n": 10000, "dx": 1, "dz": 5, "k": 4, "S": 200, "theiler": 0},
        # the tests of a search's first round over the sources: one conditioning variable
        {"name": "test n9995 dz1", "kind": "test", "n": 9995, "dx": 1, "dz": 1, "k": 4, "S": 200, "theiler": 0},
        # the first tests of a search: nothing to condition on yet
        {"name": "test n9995 dz0", "kind": "test", "n": 9995, "dx": 1, "dz": 0, "k": 4, "S": 200, "theiler": 0},
        # an omnibus test: the selected sources together given the target's past
        {"name": "omnibus n9995 dx4 dz1", "kind": "test", "n": 9995, "dx": 4, "dz": 1, "k": 4, "S": 200, "theiler": 0},
        # a long recording with autocorrelation: fewer surrogates, a Theiler window
        {"name": "test n30011 dz4 theiler", "kind": "test", "n": 30011, "dx": 1, "dz": 4, "k": 4, "S": 100,
         "theiler": 20},
        # a burst of a serving mix: unrelated tests of uneven length and conditioning dimension
        {"name": "served 32 requests", "kind": "served", "requests": 32, "n_max": 10000, "S": 200, "k": 4},
        # the whole call: every target of a small network
        {"name": "network P8 T3000", "kind": "network", "P": 8, "T": 3000, "S": 200, "k": 4},
        # the Gaussian estimator at a search's size: one covariance, one round of candidates
        {"name": "gauss D51 n9995 sets45", "kind": "gauss", "D": 51, "n": 9995, "sets": 45},
        # the largest covariance the library takes, a long recording
        {"name": "gauss D512 n1000000", "kind": "gauss", "D": 512, "n": 1000000, "sets": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["estimate", "estimate", "test", "test", "test", "test", "hosttest", "served", "network",
                       "search", "gauss", "gauss"])
    k = rng.choice([4, 4, 4, 4, 3, 8])
    if kind == "estimate":
        return {"kind": kind, "n": _log(rng, 500, 20000), "dx": rng.choice([1, 1, 1, 2]), "dz": rng.randint(0, 15),
                "k": k, "theiler": rng.choice([0, 0, 5])}
    if kind == "test":
        dz = rng.choice([0, 1, 1, 2, 3, 4, 5, 6, 8, 11, 15])
        dx = rng.choice([1, 1, 1, 1, 2, 3, 4]) if dz else 1
        n = _log(rng, 600, 10000) if dx > 1 or dz == 0 else _log(rng, 600, 30000)
        return {"kind": kind, "n": n, "dx": dx, "dz": dz, "k": k, "S": rng.choice([50, 99, 100, 200, 200, 200]),
                "theiler": rng.choice([0, 0, 0, 7, 20])}
    if kind == "hosttest":
        reps = rng.choice([1, 1, 10])
        return {"kind": kind, "n": _log(rng, 60, 600) * 10 + (rng.randint(0, 9) if reps == 1 else 0), "dx": 1,
                "dz": rng.randint(1, 8), "k": k, "S": rng.choice([50, 100, 200]), "reps": reps}
    if kind == "served":
        return {"kind": kind, "requests": rng.randint(4, 40), "n_max": _log(rng, 1000, 10000), "S": 200, "k": k}
    if kind == "network":
        return {"kind": kind, "P": rng.randint(4, 8), "T": _log(rng, 800, 3000), "S": rng.choice([100, 200]), "k": 4}
    if kind == "search":
        return {"kind": kind, "P": rng.randint(3, 10), "T": _log(rng, 800, 5000), "S": rng.choice([100, 200]), "k": 4}
    sets = rng.choice([0, 5, 45])
    D = _log(rng, 8, 512)
    return {"kind": kind, "D": D, "n": _log(rng, 1000, 1000000), "sets": sets}


# ---------------------------------------------------------------- inputs
def _var_series(g, P, T):
    """A stable linear VAR with self-coupling 0.4 and up to three sources per process at lags 1..5,
    unit noise, [P][T] float32."""
    m = min(3, P - 1)
    src = np.stack([g.choice(np.delete(np.arange(P), i), size=m, replace=False) for i in range(P)])
    lag = g.integers(1, MAX_LAG + 1, size=(P, m))
    coef = g.uniform(0.1, 0.22, size=(P, m))
    burn = 200
    x = np.zeros((burn + T, P))
    noise = g.standard_normal((burn + T, P))
    for t in range(MAX_LAG, burn + T):
        x[t] = 0.4 * x[t - 1] + (coef * x[t - lag, src]).sum(1) + noise[t]
    return np.ascontiguousarray(x[burn:].T.astype(np.float32)), src, lag


def _clm_series(g, P, T):
    """Coupled logistic maps on a random graph (coupling 0.5 over three sources, noise s.d. 0.1),
    [P][T] float32."""
    m = min(3, P - 1)
    src = g.integers(0, P, size=(P, m))
    lag = g.integers(1, MAX_LAG + 1, size=(P, m))
    burn = 200
    f = np.zeros((burn + T, P))
    x = np.zeros((burn + T, P))
    x[:MAX_LAG] = g.random((MAX_LAG, P))
    f[:MAX_LAG] = 4 * x[:MAX_LAG] * (1 - x[:MAX_LAG])
    noise = 0.1 * g.standard_normal((burn + T, P))
    for t in range(MAX_LAG, burn + T):
        v = (0.5 * f[t - 1] + 0.5 * f[t - lag, src].mean(1) + noise[t]) % 1.0
        x[t] = v
        f[t] = 4 * v * (1 - v)
    return np.ascontiguousarray(x[burn:].T.astype(np.float32))


def _triple(case, seed):
    """X [dx][n], Y [1][n], Z [dz][n] (None without Z) as float32 host arrays: for one Z variable or
    fewer and a single estimate a Gaussian triple, else lagged variables of a VAR: Y a process's
    present, Z its past and then other processes' pasts, X its sources at their lags."""
    g = np.random.default_rng([seed, case["n"]])
    n, dx, dz = case["n"], case["dx"], case["dz"]
    if case["kind"] == "estimate" and dx == 1 and dz <= 1:
        z, u, w = g.standard_normal((3, n))
        s = math.sqrt(1 - 0.3 ** 2)
        x, y = 0.3 * z + s * u, 0.3 * z + s * (0.6 * u + 0.8 * w)
        f = lambda a: np.ascontiguousarray(a.astype(np.float32)[None])  # noqa: E731
        return f(x), f(y), f(z) if dz else None
    series, src, lag = _var_series(g, 10, n + MAX_LAG)
    col = lambda node, lg: series[node, MAX_LAG - lg:MAX_LAG - lg + n]  # noqa: E731
    zv = [(0, lg) for lg in range(1, MAX_LAG + 1)] + [(p, lg) for p in range(4, 10) for lg in (1, 3)]
    xv = [(int(src[0, j]), int(lag[0, j])) for j in range(3)] + [(9, 5)]
    stack = lambda v: np.ascontiguousarray(np.stack([col(*q) for q in v]))  # noqa: E731
    return stack(xv[:dx]), stack([(0, 0)]), stack(zv[:dz]) if dz else None


def _requests(case, seed):
    g = np.random.default_rng([seed, 77])
    reqs = []
    for r in range(case["requests"]):
        n = max(300, int(case["n_max"] * (0.1, 0.3, 1.0)[r % 3]))
        dz = 1 + (r * 7 + 3) % 15
        nodes = g.permutation(100)[:2 + dz].astype(np.int32)
        lags = np.concatenate([[int(g.integers(1, 6))], [0], g.integers(1, 6, size=dz)]).astype(np.int32)
        reqs.append(dict(nodes=nodes, lags=lags, dx=1, dy=1, dz=dz, t0=MAX_LAG, n=n, k=case["k"], S=case["S"],
                         seed=seed, cand=r))
    return reqs


def _gauss_sets(case, seed):
    """A greedy round's (X, Y, Z) index sets: every candidate in turn as X, variable 0 as Y and the
    same conditioning set."""
    g = np.random.default_rng([seed, 5])
    dz = min(6, case["D"] - 2)
    order = g.permutation(np.arange(1, case["D"]))
    z = [int(v) for v in order[:dz]]
    rest = [int(v) for v in order[dz:]]
    return [([rest[j % len(rest)]], [0], z) for j in range(case["sets"])]


def _gauss_data(case, seed):
    """Correlated Gaussian columns with means of their own, [D][n] float32 on the device."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    D, n = case["D"], case["n"]
    v = torch.empty(D, n, dtype=torch.float32, device="cuda").normal_(generator=gen)
    common = torch.empty(n, dtype=torch.float32, device="cuda").normal_(generator=gen)
    mean = torch.empty(D, 1, dtype=torch.float32, device="cuda").normal_(generator=gen)
    return v.add_(0.5 * common).add_(mean)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("estimate", "test"):
        X, Y, Z = _triple(case, seed)
        dev = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
        out = torch.zeros(1 + case.get("S", 0), dtype=torch.float64, device="cuda")
        return {"case": case, "seed": seed, "X": dev(X), "Y": dev(Y), "Z": dev(Z), "out": out}
    if kind == "hosttest":
        X, Y, Z = _triple(case, seed)
        return {"case": case, "seed": seed, "X": X, "Y": Y, "Z": Z}
    if kind == "served":
        series = _clm_series(np.random.default_rng([seed, 3]), 100, case["n_max"] + MAX_LAG)
        return {"case": case, "sid": mte.mte_series_register(series), "reqs": _requests(case, seed)}
    if kind in ("network", "search"):
        series, _, _ = _var_series(np.random.default_rng([seed, 9]), case["P"], case["T"])
        return {"case": case, "seed": seed, "series": series}
    D = case["D"]
    return {"case": case, "V": _gauss_data(case, seed), "sets": _gauss_sets(case, seed),
            "cov": torch.zeros(D, D, dtype=torch.float64, device="cuda")}


# ---------------------------------------------------------------- one pass
def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "estimate":
        if c["theiler"]:
            mte.cmi_ksg_surrogates_dev(state["X"], state["Y"], state["Z"], c["k"], 0, 0, 0, state["out"],
                                       theiler=c["theiler"])
        else:
            mte.cmi_ksg_dev(state["X"], state["Y"], state["Z"], c["k"], state["out"])
        return {"estimate": state["out"]}
    if kind == "test":
        mte.cmi_ksg_surrogates_dev(state["X"], state["Y"], state["Z"], c["k"], c["S"], state["seed"], 0,
                                   state["out"], theiler=c["theiler"])
        return {"estimate": state["out"][:1], "surrogates": state["out"][1:]}
    if kind == "hosttest":
        if c["reps"] > 1:
            cmi, surr = mte.cmi_ksg_surrogates_rep(state["X"], state["Y"], state["Z"], k=c["k"], S=c["S"],
                                                   R=c["reps"], seed=state["seed"])
        else:
            cmi, surr = mte.cmi_ksg_surrogates(state["X"], state["Y"], state["Z"], k=c["k"], S=c["S"],
                                               seed=state["seed"])
        return {"estimate": cmi, "surrogates": surr}
    if kind == "served":
        tickets = [mte.mte_submit(state["sid"], **q) for q in state["reqs"]]
        got = [mte.mte_wait(t, c["S"]) for t in tickets]
        return {"estimate": np.array([e for e, _ in got]), "surrogates": np.stack([s for _, s in got])}
    if kind == "network":
        adj, summ = mte.mte_infer_network(state["series"], max_lag_sources=MAX_LAG, alpha=0.05, alpha_fdr=0.05,
                                          k=c["k"], S=c["S"], seed=state["seed"])
        return {"adjacency": adj, "te": np.array([s["omnibus_te"] for s in summ]),
                "p": np.array([s["omnibus_p"] for s in summ]),
                "counts": np.array([[s["n_target_past"], s["n_sources_tested"], s["n_estimates"]] for s in summ])}
    if kind == "search":
        r = mte.mte_select_sources(state["series"], 0, list(range(1, c["P"])), max_lag_sources=MAX_LAG, alpha=0.05,
                                   k=c["k"], S=c["S"], seed=state["seed"])
        var = [v for key in ("target_past", "sources_before_omnibus") for v in r[key]]
        return {"selected": np.array([[v[0], v[1]] for v in var] + [[len(r["target_past"]), r["n_estimates"]]]),
                "cmi": np.array([v[2] for v in var] + [r["omnibus_te"]]),
                "p": np.array([v[3] for v in var] + [r["omnibus_p"]])}
    mte.mte_gauss_covariance_dev(state["V"], state["cov"])
    if not state["sets"]:
        return {"cov": state["cov"]}
    return {"cov": state["cov"], "cmi": mte.mte_gauss_cmi_sets(state["cov"], state["sets"])}


# ---------------------------------------------------------------- work
def _test_work(n, dx, dz, k, est):
    """A test reads its columns and writes its estimates; every (row, estimate) pair needs at least
    the joint distances of its k neighbours (a subtraction and a maximum per variable) and the three
    digamma terms."""
    return {"bytes": 4.0 * n * (dx + 1 + dz) + 8.0 * est, "flops": float(n) * est * (2 * k * (dx + 1 + dz) + 4)}


def work(case):
    kind = case["kind"]
    if kind in ("estimate", "test", "hosttest"):
        return _test_work(case["n"], case["dx"], case["dz"], case["k"], 1 + case.get("S", 0))
    if kind == "served":
        parts = [_test_work(q["n"], 1, q["dz"], q["k"], 1 + q["S"]) for q in _requests(case, 0)]
        return {key: sum(p[key] for p in parts) for key in ("bytes", "flops")}
    if kind in ("network", "search"):
        # per target at least one round over its own lags and two over the sources' lags
        P, T = case["P"], case["T"]
        n, targets = T - MAX_LAG, P if kind == "network" else 1
        est = targets * (MAX_LAG + 2 * (P - 1) * MAX_LAG) * (1 + case["S"])
        return {"bytes": 4.0 * P * T + 40.0 * targets, "flops": float(n) * est * (2 * case["k"] * 3 + 4)}
    D, n = case["D"], case["n"]
    return {"bytes": 4.0 * D * n + 8.0 * D * D, "flops": float(D) * (D + 1) * n}


# ---------------------------------------------------------------- exact values
def _ksg_exact(X, Y, Z, k, w):
    """The estimate from its definition, all pairs: distances are single-precision differences,
    radii and strict counts follow, the digamma terms are summed in 64 bits."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    put = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    X, Y, Z = put(X), put(Y), put(Z)
    n = X.shape[1]
    rows = torch.arange(n, device=dev)
    total = torch.zeros((), dtype=torch.float64, device=dev)
    step = max(1, min(n, 40_000_000 // n))
    psi = lambda v: torch.special.digamma(v.double() + 1)  # noqa: E731

    def dist(V, i):
        d = (V[0, i, None] - V[0][None, :]).abs()
        for c in range(1, V.shape[0]):
            d = torch.maximum(d, (V[c, i, None] - V[c][None, :]).abs())
        return d

    for a in range(0, n, step):
        i = rows[a:a + step]
        near = (i[:, None] - rows[None, :]).abs() <= w
        inf = float("inf")
        dx, dy = dist(X, i).masked_fill_(near, inf), dist(Y, i).masked_fill_(near, inf)
        if Z is not None:
            dz = dist(Z, i)
            dx, dy = torch.maximum(dx, dz), torch.maximum(dy, dz)
        eps = torch.topk(torch.maximum(dx, dy), k, dim=1, largest=False).values[:, -1:]
        if Z is not None:
            nz = (dz.masked_fill_(near, inf) < eps).sum(1)
        else:
            nz = n - near.sum(1)
        total += (psi((dx < eps).sum(1)) + psi((dy < eps).sum(1)) - psi(nz)).sum()
    return float(torch.special.digamma(torch.tensor(float(k), dtype=torch.float64))) - float(total) / n


def exact(case, seed):
    kind = case["kind"]
    if kind in ("estimate", "test", "hosttest"):
        v = _ksg_exact(*_triple(case, seed), case["k"], case.get("theiler", 0))
        if kind == "hosttest":
            return {"estimate": v, "surrogates": None}
        est = torch.tensor([v], dtype=torch.float64)
        return {"estimate": est} if kind == "estimate" else {"estimate": est, "surrogates": None}
    if kind == "served":
        series = _clm_series(np.random.default_rng([seed, 3]), 100, case["n_max"] + MAX_LAG)
        got = []
        for q in _requests(case, seed):
            v = np.stack([series[p, q["t0"] - lg:q["t0"] - lg + q["n"]] for p, lg in zip(q["nodes"], q["lags"])])
            got.append(_ksg_exact(v[:1], v[1:2], v[2:], q["k"], 0))
        return {"estimate": np.array(got), "surrogates": None}
    if kind in ("network", "search"):
        return None
    V = _gauss_data(case, seed)
    D, n = V.shape
    mean = V.sum(1, keepdim=True, dtype=torch.float64) / n
    cov = torch.zeros(D, D, dtype=torch.float64, device=V.device)
    for a in range(0, n, 65536):
        b = V[:, a:a + 65536].double() - mean
        cov += b @ b.T
    cov /= n
    sets = _gauss_sets(case, seed)
    if not sets:
        return {"cov": cov}
    h = cov.cpu()
    logdet = lambda v: float(torch.linalg.slogdet(h[v][:, v]).logabsdet) if v else 0.0  # noqa: E731
    cmi = [0.5 * (logdet(x + z) + logdet(y + z) - logdet(z) - logdet(x + y + z)) for x, y, z in sets]
    return {"cov": cov, "cmi": np.array(cmi)}
