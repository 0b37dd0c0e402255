"""Jobs without Z, with one X and one Y column, walk the ranks of y.

No neighbour lists are built: a row's neighbours in y are the ranks next to its
own, and n_x and n_y are ranges of the sorted columns.  Radii, counts and
estimates must be the oracle's and the all-pairs kernel's bit for bit."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth
from test_gpu_parity import check_against_oracle, oracle_estimates

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# fewer rows than a step, one step, more than the pads; ties and wide values
@pytest.mark.parametrize("n,k,kind,S", [(2, 1, "normal", 8), (7, 4, "grid", 8), (9, 8, "normal", 8),
                                        (17, 16, "dup", 8), (64, 4, "grid", 63), (65, 4, "normal", 70),
                                        (1000, 4, "dup", 9), (1999, 5, "wide", 9), (700, 4, "tiny", 200)])
def test_walk_parity(monkeypatch, n, k, kind, S):
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    X, Y, _ = synth.random_points(n, (1, 1, 0), seed=n + k, kind=kind)
    say("walk", n, k, kind, S)
    check_against_oracle(X, Y, None, k, S)


@pytest.mark.parametrize("n,w", [(300, 1), (300, 140), (1000, 20)])
def test_walk_theiler(monkeypatch, n, w):
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    X, Y, _ = synth.random_points(n, (1, 1, 0), seed=n + w, kind="normal")
    say("walk, window", n, w)
    cmi, eps, cx, cy, cz = mte.cmi_ksg_diag(X, Y, None, 4, 9, 3, 1, theiler=w)
    for e, (v, re, ra, rb, rc) in enumerate(oracle_estimates(X, Y, None, 4, 9, 3, 1, theiler=w)):
        assert np.array_equal(eps[e], re) and np.array_equal(cx[e], ra)
        assert np.array_equal(cy[e], rb) and np.array_equal(cz[e], rc)
        assert abs(cmi[e] - v) < 1e-9


@pytest.mark.parametrize("n", [9984, 16384])
def test_walk_sizes(monkeypatch, n):
    X, Y, _ = synth.random_points(n, (1, 1, 0), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        say("walk sizes", n, mode)
        out[mode] = mte.cmi_ksg_diag(X, Y, None, 4, 66, 5, 1)
    for a, b in zip(out["brute"], out["list"]):
        assert np.array_equal(a, b)
