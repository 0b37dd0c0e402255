"""The tuner times only the knobs that a shape's kernels read; the others keep their defaults."""

import sys

import pytest
import torch

import paper_1902_06828_amd as mte
import synth

pytestmark = pytest.mark.gpu


# a walk builds and scans no lists, and its permutation waits for ranks; counts by ranks of z scan
# lists, and their permutation waits too
@pytest.mark.parametrize("dz,kept", [(0, {"build_rows": 0, "coop_lanes": 4, "scan_step": 8, "perm_cu": 2}),
                                     (1, {"perm_cu": 2})])
def test_knobs_without_effect_keep_their_defaults(monkeypatch, tmp_path, dz, kept):
    monkeypatch.setenv("MTE_TUNE_FILE", str(tmp_path / "tune.txt"))
    monkeypatch.delenv("MTE_TUNE", raising=False)
    mte.mte_shutdown()                      # the next call starts anew
    # every candidate in reach of the tuning, several shapes: one of them picked by noise shows
    monkeypatch.setenv("MTE_TUNE_BUDGET_MS", "2000")
    for n in range(400, 1000, 100):
        X, Y, Z = [None if a is None else torch.from_numpy(a).cuda()
                   for a in synth.random_points(n, (1, 1, dz), seed=n)]
        out = torch.zeros(41, dtype=torch.float64, device="cuda")
        print("tuning", n, dz, flush=True)
        sys.stdout.flush()
        mte.cmi_ksg_surrogates_dev(X, Y, Z, 4, 40, 1, 0, out)
    torch.cuda.synchronize()
    rep = mte.mte_tune_report()
    print(rep, flush=True)
    assert len(rep) == 6
    for r in rep:
        assert {k: r[k] for k in kept} == kept
    mte.mte_shutdown()
