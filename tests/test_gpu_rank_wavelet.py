"""Counts in wavelet matrices and permutations by table swaps.

Sets with one Z column take n_xz of a one-X-column job without a window from a
wavelet matrix per estimate, up to the rows that fit a block's LDS; launches of
many estimates permute by swaps of a table in LDS.  Radii, counts and surrogates
must be the oracle's, and those of the all-pairs kernel, bit for bit."""

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


# one row, one 64-row block and its neighbours, a power of two (one bit more
# than the largest rank needs), several blocks per wave; values with ties
@pytest.mark.parametrize("n,k,kind", [(2, 1, "normal"), (63, 4, "grid"), (64, 4, "normal"), (65, 4, "dup"),
                                      (128, 3, "grid"), (1024, 4, "tiny"), (1025, 8, "normal"), (2047, 4, "wide")])
def test_wavelet_counts_parity(monkeypatch, n, k, kind):
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    X, Y, Z = synth.random_points(n, (1, 1, 1), seed=n + k, kind=kind)
    say("wavelet counts", n, k, kind)
    check_against_oracle(X, Y, Z, k, 9)


# the largest sizes of one and of two blocks per CU, the last that fits LDS
# and the first that does not (counted over rank ranges)
@pytest.mark.parametrize("n", [9984, 16384, 20990, 21100])
def test_wavelet_counts_sizes(monkeypatch, n):
    X, Y, Z = synth.random_points(n, (1, 1, 1), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        say("wavelet sizes, N", n, mode)
        out[mode] = mte.cmi_ksg_diag(X, Y, Z, 4, 8, 5, 1)
    for a, b in zip(out["brute"], out["list"]):
        assert np.array_equal(a, b)


# permutations of a few rows, odd and even sizes, the largest table and the
# first size above it, with enough estimates for the table form; within
# replications too
@pytest.mark.parametrize("n,R,S", [(16, 1, 600), (999, 1, 600), (1000, 10, 700), (4096, 1, 520), (16384, 1, 513),
                                   (16385, 1, 513)])
def test_table_permutation(monkeypatch, n, R, S):
    X, Y, Z = synth.random_points(n, (1, 1, 2), seed=n)
    out = {}
    for mode in ("brute", "list"):
        monkeypatch.setenv("MTE_FORCE_MODE", mode)
        say("table permutation", n, R, S, mode)
        if R > 1:
            out[mode] = mte.cmi_ksg_surrogates_rep(X, Y, Z, k=4, S=S, R=R, seed=3, mode="within")
        else:
            out[mode] = mte.cmi_ksg_surrogates(X, Y, Z, k=4, S=S, seed=3)
    assert out["brute"][0] == out["list"][0] and np.array_equal(out["brute"][1], out["list"][1])
