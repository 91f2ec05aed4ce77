"""The batched launches: instances at the edges of their classes of sizes, the
tuned plan of a batch whose small
instances go elsewhere, and the launch's own scheduling at sizes that now run
in registers (forced here with APX_BATCH_WPC).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu


def _s(n, seed=0):
    pts = synth.gaussian_2d(n=n, k=4, seed=n + seed) if n < 200 else synth.gaussian_mixture(n=n, d=8, k=7, seed=n + seed)
    return apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=n)[0]


def _solve(Ss, **kw):
    R, A = ([apx.empty_matrix(S.shape[0]) for S in Ss] for _ in "RA")
    idx, res = apx.ap_solve_batched(Ss, R, A, damping=0.9, max_iter=40, conv_iter=0)
    return idx, R, A, res


@pytest.mark.parametrize("large,small", [([4000, 3500], [300] * 30), ([6000], [50, 700]), ([3073, 3200, 5000, 3100], [64] * 60)])
def test_a_tuned_plan_serves_the_streamed_part(large, small, monkeypatch):
    """A plan tuned for a mixed batch is the one its large instances run with,
    beside the small ones and alone."""
    Ss = [_s(n) for n in large + small]
    apx.apx_tune_clear()
    default = _solve(Ss)
    try:
        pick = apx.apx_autotune_batched(large + small)
        mixed, alone = _solve(Ss), _solve(Ss[:len(large)])
    finally:
        apx.apx_tune_clear()
    print("pick", pick, flush=True)
    monkeypatch.setenv("APX_BATCH_WPC", str(pick["wpc"]))
    monkeypatch.setenv("APX_BATCH_MIN_ROWS", str(pick["min_rows"]))
    ref = _solve(Ss[:len(large)])
    same_as_default = all(torch.equal(ref[1][j], default[1][j]) for j in range(len(large)))
    print("plan differs from the default:", not same_as_default, flush=True)
    for j in range(len(large)):
        for x in (0, 1, 2):
            assert torch.equal(mixed[x][j], ref[x][j]) and torch.equal(alone[x][j], ref[x][j])


@pytest.mark.parametrize("wpc", [1, 4])
def test_more_instances_than_workgroups(wpc, monkeypatch):
    """Queues of one-workgroup teams: every instance equals its oracle run."""
    count = 256 * wpc + 40
    rng = np.random.default_rng(wpc)
    Ss = [_s(int(n), seed=j) for j, n in enumerate(rng.integers(8, 60, count))]
    monkeypatch.setenv("APX_BATCH_WPC", str(wpc))
    idxs, res = apx.ap_solve_batched(Ss, damping=0.9, max_iter=300, conv_iter=15)
    for S, idx, r in zip(Ss, idxs, res):
        ref = oracle.ap(S.cpu().numpy().astype(np.float64), 0.9, 300, 15)
        assert r.iterations == ref.iterations and np.array_equal(idx.cpu().numpy(), ref.idx)


@pytest.mark.parametrize("sizes", [[40, 700, 300], [1500, 100], list(range(20, 500, 37)), [3000, 2900, 64]])
def test_teams_at_small_sizes(sizes, monkeypatch):
    Ss = [_s(n) for n in sizes]
    monkeypatch.setenv("APX_BATCH_WPC", "2")
    idxs, res = apx.ap_solve_batched(Ss, damping=0.9, max_iter=400, conv_iter=15)
    for S, idx, r in zip(Ss, idxs, res):
        ref = oracle.ap(S.cpu().numpy().astype(np.float64), 0.9, 400, 15)
        assert r.iterations == ref.iterations and r.converged == ref.converged
        assert np.array_equal(idx.cpu().numpy(), ref.idx)


def test_edges_of_the_classes():
    """Instances at the limits of the register launches and beyond, in one call:
    each as ap_solve gives it (the streamed one to rounding)."""
    sizes = [2048, 1024, 3072, 2049, 1025, 3073, 2]
    Ss = [_s(n) if n > 2 else apx.to_matrix(torch.tensor([[-0.5, -1.0], [-1.5, -0.25]])) for n in sizes]
    idx, R, A, res = _solve(Ss)
    for j, n in enumerate(sizes):
        r, a = apx.empty_matrix(n), apx.empty_matrix(n)
        one, out = apx.ap_solve(Ss[j], r, a, 0.9, 40, 0)
        assert torch.equal(idx[j], one) and res[j].n_exemplars == out.n_exemplars
        if n <= 3072:
            assert torch.equal(R[j], r) and torch.equal(A[j], a) and res[j] == out
        else:
            torch.testing.assert_close(R[j], r, rtol=0, atol=1e-4 * float(Ss[j].max() - Ss[j].min()))
