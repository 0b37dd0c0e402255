"""The sums over rows in one launch (few row chunks, or many estimates) and in
two: the estimates are the all-pairs kernel's bit for bit on both sides of each
limit (64 and 512 chunks of 64 rows, 64 estimates)."""

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,n,S", [("solo", 5, 0), ("solo", 64, 0), ("solo", 65, 0), ("solo", 4096, 0),
                                      ("solo", 4097, 0), ("list", 4097, 62), ("list", 4097, 63),
                                      ("list", 32768, 63), ("list", 32769, 63)])
def test_sums_are_the_same_bits(monkeypatch, mode, n, S):
    X, Y, Z = synth.random_points(n, (1, 1, 1), seed=n, kind="normal")
    out = []
    for m in ("brute", mode):
        monkeypatch.setenv("MTE_FORCE_MODE", m)
        print("sums", m, n, S, flush=True)
        out.append(mte.cmi_ksg_diag(X, Y, Z, 4, S, 5, 1)[0])
    assert np.array_equal(out[0], out[1])
