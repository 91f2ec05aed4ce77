"""Similarities of -inf (pairs that may not be joined) in the one-launch solve.

The launched passes (``apx_set_graphs(False)``) are the reference: R, A,
labels and sums must be the same, infinities and NaNs included.
"""
import math

import pytest
import torch

import paper_0910_1650_amd as apx

pytestmark = pytest.mark.gpu


def _neighbours_only(n, k, seed):
    """s finite for the k nearest neighbours of a point and its preference, -inf elsewhere."""
    X = torch.rand(n, 2, generator=torch.Generator().manual_seed(seed))
    D = -(X[:, None, :] - X[None, :, :]).square().sum(-1)
    D.fill_diagonal_(-math.inf)
    S = torch.full((n, n), -math.inf)
    near = D.topk(k, dim=1).indices
    S.scatter_(1, near, D.gather(1, near))
    S.fill_diagonal_(float(D[D > -math.inf].median()))
    return S


def _solve(S, on, start=None, **kw):
    apx.apx_set_graphs(on)
    try:
        R, A = (apx.to_matrix(m) for m in start) if start else (apx.empty_matrix(S.shape[0]) for _ in "RA")
        idx, res = apx.ap_solve(S, R, A, **kw)
    finally:
        apx.apx_set_graphs(True)
    return idx.cpu(), res, R.cpu(), A.cpu()


def _same(S, **kw):
    a, b = _solve(S, True, **kw), _solve(S, False, **kw)
    for x, y in zip(a[2:], b[2:]):
        torch.testing.assert_close(x, y, rtol=0, atol=0, equal_nan=True)
    assert torch.equal(a[0], b[0])
    assert a[1].n_exemplars == b[1].n_exemplars and a[1].iterations == b[1].iterations
    for x, y in ((a[1].dpsim, b[1].dpsim), (a[1].expref, b[1].expref)):
        assert x == y or (math.isnan(x) and math.isnan(y))
    return a


@pytest.mark.parametrize("n", [40, 300, 700, 2400])
def test_points_without_a_reachable_exemplar(n):
    """A point at -inf from every exemplar is labelled with the lowest one
    (-1 only where there is no exemplar at all)."""
    S = _neighbours_only(n, 4, n)
    M = apx.to_matrix(S)
    cut_off = 0
    for it in (3, 5, 8, 13):
        idx, res, _, _ = _same(M, damping=0.5, max_iter=it, conv_iter=0)
        ex = torch.nonzero(idx == torch.arange(n, dtype=torch.int32)).flatten()
        if len(ex) == 0:
            continue
        lost = (S[:, ex] == -math.inf).all(1)
        assert (idx[lost] == int(ex[0])).all()
        cut_off += int(lost.sum())
    assert cut_off > 0


@pytest.mark.parametrize("n", [40, 700, 2400])
@pytest.mark.parametrize("damping", [0.0, 0.5])
def test_points_with_one_neighbour_and_no_preference(n, damping):
    """Preference -inf and a single neighbour: r(i,k) of that neighbour is
    +inf, so its column's sum is too, and availabilities are min(0, inf - inf);
    without damping 0 * inf makes further NaNs; a run can start from such messages."""
    S = _neighbours_only(n, 4, n)
    lone = torch.arange(0, n, 5)
    best = S.clone().fill_diagonal_(-math.inf).max(1)
    S[lone] = -math.inf
    S[lone, best.indices[lone]] = best.values[lone]
    M = apx.to_matrix(S)
    for it in (1, 2, 5, 13):
        _, _, R, A = _same(M, damping=damping, max_iter=it, conv_iter=0)
        if damping:
            assert (R[lone] == math.inf).any(1).all()
            _same(M, warm=apx.APX_WARM_AR, start=(R, A), damping=damping, max_iter=3, conv_iter=0)
