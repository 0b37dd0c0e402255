"""Requests of one or a few estimates that share a (Y, Z) sample.

Batched by the request loop they share the sample's lists; each must return what a call of its own
returns, bit for bit, and a batch must not take memory that its estimates do not need."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte

pytestmark = pytest.mark.gpu

L = 5


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def burst(series, jobs, n, dx, dz, k, S, theiler=0):
    """`jobs` requests: Y is node 0, Z nodes 1..dz, X further nodes at lag 1 + j % 5."""
    P = series.shape[0]
    sid = mte.mte_series_register(series)
    try:
        mte.mte_serve_get_stats(reset=True)
        tickets, cols = [], []
        for j in range(jobs):
            xn = [1 + dz + (j + q) % (P - 1 - dz) for q in range(dx)]
            nodes = np.array(xn + [0] + list(range(1, 1 + dz)), np.int32)
            lags = np.array([1 + j % L] * dx + [0] + [1 + q % L for q in range(dz)], np.int32)
            cols.append([series[p, L - g:L - g + n] for p, g in zip(nodes, lags)])
            tickets.append(mte.mte_submit(sid, nodes=nodes, lags=lags, dx=dx, dy=1, dz=dz, t0=L, n=n, k=k, S=S,
                                          seed=7, cand=j, theiler=theiler))
        got = [mte.mte_wait(t, S) for t in tickets]
        peak = mte.mte_serve_get_stats()["peak_bytes_in_use"]
    finally:
        mte.mte_series_release(sid)
    return got, [np.ascontiguousarray(np.stack(c)) for c in cols], peak


def series_of(P, n, seed):
    g = np.random.default_rng(seed)
    x = g.standard_normal((P, n + L)).astype(np.float32)
    x[1:] += 0.5 * x[0]
    return x


def test_one_estimate_with_several_x_columns_takes_no_lists_of_its_own():
    n, jobs = 3000, 96
    say("one estimate each, 2 X columns", n, jobs)
    got, cols, peak = burst(series_of(20, n, 1), jobs, n, 2, 1, 4, 0)
    for (v, _), c in list(zip(got, cols))[::7]:
        assert v == mte.cmi_ksg(c[:2], c[2:3], c[3:], 4)
    # three batches in flight, each with the sample's lists (whole, 8 bytes an entry), and 1 KB a job's row
    say("peak", peak)
    assert peak < 3 * (8 * n * (n + 64)) + 1024 * n * jobs
