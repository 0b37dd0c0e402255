"""Replications on the forms that use ranks: exchanged sides and the rank walk, both shuffle modes.

The estimate and every surrogate must be the oracle's over the permutation's source rows; 520
estimates take the permutation by table swaps (within replications)."""

import sys

import numpy as np
import pytest

import paper_1902_06828_amd as mte
import synth
from oracle import cksg, perm

pytestmark = pytest.mark.gpu

TOL = 1e-9


@pytest.mark.parametrize("n,R,dx,dz,mode,S", [(1200, 6, 3, 1, "within", 12), (1200, 6, 2, 1, "replications", 12),
                                              (1001, 7, 4, 1, "within", 9), (600, 10, 2, 1, "within", 519),
                                              (700, 7, 1, 0, "within", 519), (700, 7, 1, 0, "replications", 12)])
def test_rank_forms_over_replications(monkeypatch, n, R, dx, dz, mode, S):
    monkeypatch.setenv("MTE_FORCE_MODE", "list")
    print("replications", n, R, dx, dz, mode, S, flush=True)
    sys.stdout.flush()
    x, y, z = synth.random_points(n, (dx, 1, dz), seed=n + dx)
    real, surr = mte.cmi_ksg_surrogates_rep(x, y, z, k=4, S=S, R=R, seed=3, cand=9, mode=mode)
    assert abs(real - cksg.cmi_ksg(x, y, z, 4)) <= TOL
    for s in range(0, S, max(1, S // 12)):
        src = perm.replication_source_rows(3, 9, s, n, R, mode)
        assert abs(surr[s] - cksg.cmi_ksg(np.ascontiguousarray(x[:, src]), y, z, 4)) <= TOL, s
