"""Requests of one or a few estimates that share a (Y, Z) sample.

Batched by the request loop they share the sample's lists; each must return what a call of its own
returns, bit for bit, and a batch must not take memory that its estimates do not need."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth

pytestmark = pytest.mark.gpu

L = 5


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def burst(series, jobs, n, dx, dz, k, S, theiler=0):
    """`jobs` requests: Y is node 0, Z nodes 1..dz, X further nodes at lag 1 + j % 5; k and S per job."""
    k, S = [list(np.broadcast_to(v, jobs)) for v in (k, S)]
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
            tickets.append(mte.mte_submit(sid, nodes=nodes, lags=lags, dx=dx, dy=1, dz=dz, t0=L, n=n, k=k[j], S=S[j],
                                          seed=7, cand=j, theiler=theiler))
        got = [mte.mte_wait(t, s) for t, s in zip(tickets, S)]
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


# one job a lane, groups that end inside a job, jobs of more than a group; two values of k, so two
# classes of lanes on one sample; ranks of z (with and without a window), lists, and the walk
@pytest.mark.parametrize("n,dx,dz,w,jobs,S", [(300, 1, 3, 0, 70, 0), (300, 2, 2, 0, 13, 9), (200, 1, 3, 0, 4, 69),
                                              (257, 1, 1, 0, 70, 0), (257, 1, 1, 3, 30, 6), (257, 1, 1, 0, 12, 19),
                                              (257, 3, 1, 0, 9, 4), (301, 1, 0, 0, 130, 0), (301, 1, 0, 5, 21, 8),
                                              (40, 1, 0, 0, 17, 12)])
def test_lanes_of_several_jobs(monkeypatch, n, dx, dz, w, jobs, S):
    ks = [4 if j % 3 else 2 for j in range(jobs)]
    say("several jobs a wave", n, dx, dz, w, jobs, S)
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    got, cols, _ = burst(series_of(20, n, n + dz), jobs, n, dx, dz, ks, S, theiler=w)
    monkeypatch.setenv("MTE_FORCE_MODE", "brute")
    for j in range(0, jobs, max(1, jobs // 11)):
        c = cols[j]
        want = mte.cmi_ksg_diag(c[:dx], c[dx:dx + 1], c[dx + 1:] if dz else None, ks[j], S, 7, j, theiler=w)[0]
        assert got[j][0] == want[0] and np.array_equal(got[j][1], want[1:])


def alone(n, dx, dz, S, theiler=0):
    """Device bytes of one request by itself."""
    sid = mte.mte_series_register(series_of(24, n, 2))
    try:
        mte.mte_serve_get_stats(reset=True)
        lags = np.array([1 + q % L for q in range(dx)] + [0] + [1 + q % L for q in range(dz)], np.int32)
        nodes = np.array(list(range(1, 1 + dx)) + [0] + list(range(1 + dx, 1 + dx + dz)), np.int32)
        mte.mte_wait(mte.mte_submit(sid, nodes=nodes, lags=lags, dx=dx, dy=1, dz=dz, t0=L, n=n, k=4, S=S, seed=1,
                                    cand=0, theiler=theiler), S)
        return mte.mte_serve_get_stats()["peak_bytes_in_use"]
    finally:
        mte.mte_series_release(sid)


# lists of m1 and m2 entries of 8 bytes, each with 16 sentinels; a pair's X twice, its counts and its
# place in the redo queue; 64 KB for tables, counters and rounding
@pytest.mark.parametrize("n,dx,dz,S,m1,m2", [(5000, 1, 3, 7, 1024, 2048), (5000, 4, 8, 7, 1024, 2048),
                                             (4000, 1, 5, 20, 1024, 2048), (4000, 2, 4, 62, 1024, 2048)])
def test_bytes_of_few_estimates(n, dx, dz, S, m1, m2):
    got = alone(n, dx, dz, S)
    row = 8 * (m1 + 16) + 8 * (m2 + 16) + 16 + 4 * (1 + dz) + (S + 1) * (8 * dx + 16.125)
    say("bytes", n, dx, dz, S, got, row * n)
    assert got < row * n + 65536


# one Z column: wavelet matrices from 64 estimates on or up to 2048 rows, rank ranges else; the
# largest sizes of one and of two wavelet blocks per CU and the last that fits
@pytest.mark.parametrize("n,S", [(2048, 7), (2049, 7), (2049, 62), (2049, 63), (9984, 63), (16384, 63), (20990, 63)])
def test_one_z_column_count_forms(monkeypatch, n, S):
    X, Y, Z = synth.random_points(n, (1, 1, 1), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        say("one Z column", n, S, mode)
        out[mode] = mte.cmi_ksg_diag(X, Y, Z, 4, S, 5, 1)
    for a, b in zip(out["brute"], out["list"]):
        assert np.array_equal(a, b)
