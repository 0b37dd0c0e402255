"""Covariance matrices at the edges of the Gram tiles (one column, a part of a
16x16 block, one column more or less than a tile, several tiles and their
diagonal) and of the row steps (fewer rows than one step, a whole step, one row
more or less), from rows that start at odd addresses."""

import numpy as np
import pytest
import torch

import paper_1902_06828_amd as mte

pytestmark = pytest.mark.gpu


def device_cov(v, first):
    """cov of the rows of v, stored `first` floats into rows of odd stride."""
    D, n = v.shape
    ld = (n + first + 2) | 1
    buf = torch.full((D, ld), float("nan"), dtype=torch.float32)
    buf[:, first:first + n] = torch.from_numpy(v)
    cov = torch.full((D, D), float("nan"), dtype=torch.float64, device="cuda")
    mte.mte_gauss_covariance_dev(buf.cuda()[:, first:], cov, n)
    return cov.cpu().numpy()


@pytest.mark.parametrize("D", [1, 16, 17, 33, 63, 64, 65, 130])
@pytest.mark.parametrize("n", [2, 31, 32, 33, 63, 65, 259, 20011])
def test_covariance_at_tile_and_step_edges(D, n):
    print("gauss tiles", D, n, flush=True)
    g = np.random.default_rng(1000 * D + n)
    v = (g.standard_normal((D, n)) + 0.5 * g.standard_normal((1, n)) + g.uniform(-30, 30, (D, 1))).astype(np.float32)
    got = device_cov(v, n % 4)
    w = v.astype(np.longdouble)
    c = w - w.mean(axis=1, keepdims=True)
    want = (c @ c.T / n).astype(np.float64)
    # N roundings of the running sum and of the products, each below half an
    # ulp of sum |a||b| <= N sd_p sd_q, and the rounding of the centered values
    sd = np.sqrt(np.diag(want))
    top = np.abs(v).max(axis=1).astype(np.float64)
    u = 2.0 ** -53
    tol = u * ((2 * n + 16) * np.outer(sd, sd) + 4 * (np.outer(top, sd) + np.outer(sd, top)) + np.outer(top, top) * u * n * n)
    assert np.all(np.abs(got - want) <= tol), np.max(np.abs(got - want) / tol)
    assert np.array_equal(got, got.T)
    # an entry has the same bits in a smaller matrix
    k = max(1, D // 2)
    assert np.array_equal(device_cov(v[D - k:], n % 3), got[D - k:, D - k:])
