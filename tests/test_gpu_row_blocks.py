"""Blocks that take all rows of an estimate (range counts, wavelet counts, one-launch sums) have as
many waves as the rows need, up to 16: sizes around one wave, around the last wave and past a block."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx,dz", [(1, 0), (1, 1), (3, 1), (1, 2)])
@pytest.mark.parametrize("n", [40, 63, 64, 65, 128, 129, 960, 961, 1023, 1024, 1025])
def test_sizes_around_the_waves(monkeypatch, n, dx, dz):
    X, Y, Z = synth.random_points(n, (dx, 1, max(dz, 1)), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        print("rows", n, dx, dz, mode, flush=True)
        sys.stdout.flush()
        out[mode] = mte.cmi_ksg_diag(X, Y, Z if dz else None, 4, 70, 3, 1)
    for a, b in zip(out["brute"], out["list"]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("dz", [0, 1])
def test_sizes_mixed_in_one_batch(monkeypatch, dz):
    sizes, P, L, S = [64, 1025, 200, 65, 961, 40] * 4, 8, 5, 9
    x = np.random.default_rng(dz).standard_normal((P, max(sizes) + L)).astype(np.float32)
    x[1:] += 0.5 * x[0]
    sid = mte.mte_series_register(x)
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    try:
        tickets = []
        for j, n in enumerate(sizes):
            print("mixed", dz, j, n, flush=True)
            nodes = np.array([1 + j % 5, 0] + [7] * dz, np.int32)
            lags = np.array([1 + j % L, 0] + [2] * dz, np.int32)
            tickets.append(mte.mte_submit(sid, nodes=nodes, lags=lags, dx=1, dy=1, dz=dz, t0=L, n=n, k=4, S=S,
                                          seed=7, cand=j))
        got = [mte.mte_wait(t, S) for t in tickets]
    finally:
        mte.mte_series_release(sid)
    monkeypatch.setenv("MTE_FORCE_MODE", "brute")
    for j, n in enumerate(sizes):
        X, Y, Z = x[1 + j % 5, L - (1 + j % L):][:n][None], x[0, L:L + n][None], x[7, L - 2:][:n][None]
        want = mte.cmi_ksg_diag(np.ascontiguousarray(X), np.ascontiguousarray(Y),
                                np.ascontiguousarray(Z) if dz else None, 4, S, 7, j)[0]
        assert got[j][0] == want[0] and np.array_equal(got[j][1], want[1:])
