"""Jobs of several X columns and one Z column, computed with the sides exchanged.

Such jobs (no Theiler window) search lists over the X columns, with Y and Z
permuted by the inverse, and count n_yz over ranks.  Radii, counts and estimates
must be the oracle's and the all-pairs kernel's bit for bit."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("caps", ["default", "2,3"])
@pytest.mark.parametrize("n,dx,k,kind", [(6, 2, 1, "normal"), (64, 2, 4, "grid"), (65, 3, 4, "dup"),
                                         (1000, 4, 4, "normal"), (777, 16, 4, "normal"), (1500, 5, 8, "wide"),
                                         (600, 2, 16, "tiny")])
def test_swapped_parity(monkeypatch, caps, n, dx, k, kind):
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    if caps != "default":
        monkeypatch.setenv("MTE_LIST_CAP", caps)
    X, Y, Z = synth.random_points(n, (dx, 1, 1), seed=n + dx, kind=kind)
    say("swapped", n, dx, k, kind, caps)
    check_against_oracle(X, Y, Z, min(k, n - 1), 9)


# both sides of the largest N (wavelet blocks in LDS), and more rows than the
# X lists hold
@pytest.mark.parametrize("n,dx", [(5000, 2), (20990, 3), (21100, 3)])
def test_swapped_sizes(monkeypatch, n, dx):
    X, Y, Z = synth.random_points(n, (dx, 1, 1), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        say("swapped sizes", n, dx, mode)
        out[mode] = mte.cmi_ksg_diag(X, Y, Z, 4, 8, 5, 1)
    for a, b in zip(out["brute"], out["list"]):
        assert np.array_equal(a, b)


def test_mixed_jobs_in_one_launch():
    # one burst of requests whose launch holds swapped jobs, jobs on the same
    # (Y, Z) sample that are not, jobs without Z and sets of several numbers
    # of Z columns (one build part each); every one equal to its own call
    series, _ = synth.var_network(8, 1200, seed=3)
    sid = mte.mte_series_register(series)
    lists = [([1], [0], [0]), ([1, 2], [0], [0]), ([1, 2, 3], [0], [4]), ([5], [0], []), ([5], [0], [1, 2]),
             ([6], [0], [1, 2, 3, 4]), ([1, 2], [0], [3, 4]), ([7], [2], [3])]
    reqs = []
    for c, (xs, ys, zs) in enumerate(lists):
        nodes = xs + ys + zs
        lags = [1 + q for q in range(len(xs))] + [0] + [1 + q % 4 for q in range(len(zs))]
        reqs.append(dict(nodes=nodes, lags=lags, dx=len(xs), dy=1, dz=len(zs), t0=5, n=1200, k=4, S=40, seed=9, cand=c))
    say("mixed launch")
    got = [mte.mte_wait(t, 40) for t in [mte.mte_submit(sid, **q) for q in reqs]]
    for q, (v, s) in zip(reqs, got):
        one = mte.mte_wait(mte.mte_submit(sid, **q), 40)
        col = lambda a, b: np.ascontiguousarray(np.stack([series[p, 5 - lg:5 - lg + 1200] for p, lg in
                                                          zip(q["nodes"][a:b], q["lags"][a:b])]))  # noqa: E731
        dx, dz = q["dx"], q["dz"]
        ref = mte.cmi_ksg_diag(col(0, dx), col(dx, dx + 1), col(dx + 1, dx + 1 + dz) if dz else None, 4, 40, 9,
                               q["cand"])[0]
        assert v == one[0] == ref[0] and np.array_equal(s, one[1]) and np.array_equal(s, ref[1:])
    mte.mte_series_release(sid)
