"""The one-launch solve (messages in registers) against the launched passes.

Both run the explicit recursion with the same row groups, so R, A, labels and
the stop iteration must agree bit for bit; ``apx_set_graphs(False)`` selects
the launched passes.  Sizes sit at the edges of its shapes: one workgroup and
two, a row group of one row and of two (n = 512, 513), full and one-column
last chunks, chunks of S in LDS (n > 2304), the largest size and the first
one beyond it (which streams either way).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu


def _s(n, d, seed):
    pts = synth.gaussian_2d(n=n, k=5, seed=seed) if d == 2 else synth.gaussian_mixture(n=n, d=d, k=12, seed=seed)
    return apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=seed)[0]


def _both(S, warm=apx.APX_COLD, start=None, **kw):
    out = []
    for on in (True, False):
        apx.apx_set_graphs(on)
        try:
            R, A = (apx.to_matrix(m) for m in start) if start else (apx.empty_matrix(S.shape[0], fill=3.0) for _ in "RA")
            idx, res = apx.ap_solve(S, R, A, warm=warm, **kw)
            out.append((idx, res, R, A))
        finally:
            apx.apx_set_graphs(True)
    a, b = out
    assert a[1].iterations == b[1].iterations and a[1].converged == b[1].converged
    assert a[1].n_exemplars == b[1].n_exemplars
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[2], b[2]) and torch.equal(a[3], b[3])
    np.testing.assert_array_equal([a[1].dpsim, a[1].expref], [b[1].dpsim, b[1].expref])
    return a


@pytest.mark.parametrize("n", [2, 8, 9, 96, 97, 256, 257, 512, 513, 1024, 1025, 2048, 2304, 2305, 2560, 2561, 2817,
                               3071, 3072, 3073])
def test_cold_equals_launched_passes(n):
    _both(_s(n, 2 if n < 300 else 16, 40 + n), damping=0.9, max_iter=400, conv_iter=15)


@pytest.mark.parametrize("n", [11, 700, 2400])
@pytest.mark.parametrize("warm", [apx.APX_WARM_A, apx.APX_WARM_AR, apx.APX_WARM_COLUMNS])
def test_warm_starts_equal_launched_passes(n, warm):
    S = _s(n, 8, 7)
    g = torch.Generator().manual_seed(n)
    col = -torch.rand(n, generator=g)
    A = col[None, :].repeat(n, 1) if warm == apx.APX_WARM_COLUMNS else -torch.rand(n, n, generator=g)
    A.diagonal().abs_()
    R = torch.randn(n, n, generator=g)
    _both(S, warm=warm, start=(R, A), damping=0.8, max_iter=300, conv_iter=15)


@pytest.mark.parametrize("kw", [dict(max_iter=1, conv_iter=15), dict(max_iter=6, conv_iter=0),
                                dict(max_iter=50, conv_iter=1), dict(max_iter=30, conv_iter=15, damping=0.0),
                                dict(max_iter=40, conv_iter=15, flags=apx.APX_RAW_LABELS),
                                dict(max_iter=40, conv_iter=3, check_every=1)])
def test_stop_rules_equal_launched_passes(kw):
    _both(_s(900, 8, 5), **{"damping": 0.9, **kw})


def test_ties_and_identical_points():
    # every off-diagonal similarity equal: the decision of each row is a tie
    n = 300
    S = torch.full((n, n), -1.0)
    S.fill_diagonal_(-0.5)
    _both(apx.to_matrix(S), damping=0.5, max_iter=20, conv_iter=5)
    _both(apx.to_matrix(torch.zeros(70, 70)), damping=0.5, max_iter=20, conv_iter=5)


@pytest.mark.parametrize("n", [130, 1500])
def test_matches_oracle(n):
    pts = synth.gaussian_mixture(n=n, d=16, k=8, seed=n)
    S, p = apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=n)
    R, A = apx.empty_matrix(n), apx.empty_matrix(n)
    idx, res = apx.ap_solve(S, R, A, 0.9, 1000, 15)
    ref = oracle.ap(S.cpu().numpy().astype(np.float64), 0.9, 1000, 15)
    assert res.converged and res.iterations == ref.iterations
    assert np.array_equal(idx.cpu().numpy(), ref.idx)


def test_padding_untouched_and_other_stream():
    n, ld = 515, 520
    S = _s(n, 4, 9)
    base = [torch.full((n, ld), 7.0, device="cuda") for _ in range(3)]
    s, r, a = (b[:, :n] for b in base)
    s.copy_(S)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        idx, _ = apx.ap_solve(s, r, a, 0.9, 300, 15)
    side.synchronize()
    assert all(bool((b[:, n:] == 7.0).all()) for b in base)
    R, A = apx.empty_matrix(n), apx.empty_matrix(n)
    idx2, _ = apx.ap_solve(S, R, A, 0.9, 300, 15)
    assert torch.equal(idx, idx2) and torch.equal(r, R) and torch.equal(a, A)


@pytest.mark.parametrize("warm", [apx.APX_COLD, apx.APX_WARM_AR])
@pytest.mark.parametrize("sizes", [[2], [60, 61, 256, 257], [3072, 1025, 1024, 768, 3, 2304], [700] * 24,
                                   list(range(40, 1024, 41)) * 2])
def test_batch_equals_single_solves(sizes, warm):
    """Every instance of a batch as ap_solve gives it, bit for bit: one that
    fits a single workgroup, both size classes in one call, a batch that fits
    the chip at once and ones that take turns."""
    Ss = [_s(n, 2 if n < 300 else 16, 300 + j) for j, n in enumerate(sizes)]
    start = [(torch.randn(n, n, generator=torch.Generator().manual_seed(n)),
              -torch.rand(n, n, generator=torch.Generator().manual_seed(n + 1))) for n in sizes]

    def fresh(j):
        return [apx.to_matrix(m) for m in start[j]]

    RA = [fresh(j) for j in range(len(sizes))]
    idxs, res = apx.ap_solve_batched(Ss, [r for r, _ in RA], [a for _, a in RA], 0.9, 60, 15, warm=warm)
    for j, S in enumerate(Ss):
        R, A = fresh(j)
        idx, one = apx.ap_solve(S, R, A, 0.9, 60, 15, warm=warm)
        assert one.iterations == res[j].iterations and one.n_exemplars == res[j].n_exemplars
        np.testing.assert_array_equal([one.dpsim, one.expref], [res[j].dpsim, res[j].expref])
        assert torch.equal(idx, idxs[j]) and torch.equal(R, RA[j][0]) and torch.equal(A, RA[j][1])


def test_streamed_batch_still_agrees(monkeypatch):
    sizes = [64, 300, 900]
    Ss = [_s(n, 16, 500 + n) for n in sizes]
    idxs, res = apx.ap_solve_batched(Ss, damping=0.9, max_iter=400, conv_iter=15)
    monkeypatch.setenv("APX_BATCH_WPC", "2")
    idx2, res2 = apx.ap_solve_batched(Ss, damping=0.9, max_iter=400, conv_iter=15)
    for a, b, r, q in zip(idxs, idx2, res, res2):
        assert torch.equal(a, b) and r.iterations == q.iterations
