"""Nearest-exemplar assignment at the edges of its kernel: one dimension, odd
and largest dimensions (318 is refused), exemplar counts around the sixteen a
workgroup takes at a time, points around a multiple of 64; the labels are the
argmin of FP64 distances, exact, with exemplars in ascending order.
"""
import numpy as np
import pytest
import torch

import paper_0910_1650_amd as apx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,L,pref", [(65, 1, 30, -0.001), (1000, 3, 200, -0.01), (1023, 127, 120, -1.0),
                                        (640, 317, 64, -5.0), (2049, 16, 1025, -0.5), (300, 5, 40, -1.0e6)])
def test_assignment_is_the_nearest_exemplar(n, d, L, pref):
    X = torch.from_numpy(np.random.default_rng(n + d).normal(size=(n, d)).astype(np.float32)).cuda()
    idx, res, ex = apx.lap_solve(X, L, seed=7, pref=pref, max_iter=200)
    assert res.n_exemplars == ex.size > 0 and np.all(np.diff(ex) > 0)
    x = X.cpu().numpy().astype(np.float64)
    dist = ((x[:, None, :] - x[None, ex, :]) ** 2).sum(2)
    want = ex[dist.argmin(1)]
    want[ex] = ex
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    np.testing.assert_allclose(res.dpsim, -dist.min(1)[np.setdiff1d(np.arange(n), ex)].sum(), rtol=1e-12)


def test_too_many_dimensions_stay_refused():
    X = torch.zeros(40, 318, device="cuda")
    X[:, 0] = torch.arange(40, device="cuda")
    with pytest.raises(apx.ApxError):
        apx.lap_solve(X, 10, seed=1)
