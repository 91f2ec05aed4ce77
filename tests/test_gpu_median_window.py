"""The median preference through the window (ap_similarity) and through the
radix select it falls back to, against numpy's median of the entries: sizes
where every key is set aside and where a sample narrows the window (512, 513),
one tile and more, points on a grid (few distinct values: one key per
interval, or several: the select), two far groups of equal size (the median
lies in the gap), identical points, a caller's workspace without room for the
set-aside keys, and data whose small distances the tie noise changes.
"""
import numpy as np
import pytest
import torch

import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu


def _median(S):
    v = S.cpu().numpy()[np.triu_indices(S.shape[0], 1)]
    m = v.size
    v = np.partition(v, [(m - 1) // 2, m // 2])
    return 0.5 * (float(v[(m - 1) // 2]) + float(v[m // 2]))


def _points(kind, n):
    rng = np.random.default_rng(n)
    if kind == "mixture":
        return synth.gaussian_mixture(n=n, d=16, k=7, seed=n).X
    if kind == "grid":
        return rng.integers(0, 12, size=(n, 2)).astype(np.float32)
    if kind == "grid6":
        return rng.integers(0, 3, size=(n, 6)).astype(np.float32)
    if kind == "gap":
        x = rng.normal(size=(n, 2)).astype(np.float32) * 0.01
        x[: n // 2] += 1000.0
        return x
    if kind == "same":
        return np.full((n, 3), 2.5, dtype=np.float32)
    return synth.gaussian_2d(n=n, k=5, seed=n).X


@pytest.mark.parametrize("kind", ["mixture", "grid", "grid6", "gap", "same", "plane"])
@pytest.mark.parametrize("n", [2, 3, 64, 181, 512, 513, 1300, 4001])
def test_median_is_exact(kind, n):
    X = torch.from_numpy(_points(kind, n)).cuda()
    S, p = apx.ap_similarity(X, noise_rel=0.0)
    assert p == _median(S)
    assert bool((S.diagonal() == np.float32(p)).all())
    # the noise changes neither the median nor any entry it need not
    S2, p2 = apx.ap_similarity(X, noise_seed=3, noise_rel=1e-12)
    assert p2 == p


@pytest.mark.parametrize("n", [300, 1300])
def test_small_workspace_takes_the_select(n):
    X = torch.from_numpy(_points("mixture", n)).cuda()
    S, p = apx.ap_similarity(X, noise_seed=3)
    # room for the select's state alone (norms, two 8192-bin histograms)
    buf = torch.empty(4 * n + (1 << 18), dtype=torch.uint8, device="cuda")
    apx.apx_set_workspace(buf)
    try:
        S2, p2 = apx.ap_similarity(X, noise_seed=3)
    finally:
        apx.apx_set_workspace(None)
    assert p2 == p and torch.equal(S, S2)


@pytest.mark.parametrize("n,d", [(5, 1), (63, 3), (64, 64), (65, 65), (200, 130)])
def test_norms_and_finite_check(n, d):
    g = torch.Generator(device="cuda").manual_seed(n)
    base = torch.randn(n, d + 3, generator=g, device="cuda")
    X = base[:, :d]
    S, _ = apx.ap_similarity(X, pref=-1.0, noise_rel=0.0)
    x = X.cpu().numpy().astype(np.float64)
    ref = -((x[:, None, :] - x[None, :, :]) ** 2).sum(2)
    off = ~np.eye(n, dtype=bool)
    bound = (d + 2) * 2.0 ** -24 * 1.01 * ((x ** 2).sum(1)[:, None] + (x ** 2).sum(1)[None, :])
    assert np.all(np.abs(S.cpu().numpy() - ref)[off] <= 2.0 * bound[off])
    base[:, d:] = float("nan")              # outside the columns: not looked at
    apx.ap_similarity(X, pref=-1.0)
    X[n - 1, d - 1] = float("inf")
    S.fill_(5.0)
    with pytest.raises(apx.ApxError):
        apx.ap_similarity(X, S=S, pref=-1.0)
    assert bool((S == 5.0).all())


def _uneven(kind, n):
    """Points whose similarities crowd: ties at the median, a far point or heavy
    tails that stretch the range, two tight clusters, a tie at zero."""
    rng = np.random.default_rng(n + 7)
    x = rng.normal(size=(n, 16))
    if kind == "binary":
        x = (x > 0).astype(float)
    elif kind == "onehot":
        x = np.eye(16)[rng.integers(0, 16, n)]
    elif kind == "halves":                    # two values only, half of the pairs each
        x = np.eye(16)[rng.integers(0, 2, n)]
    elif kind == "outlier":
        x[0] = 1.0e4
    elif kind == "heavy":
        x = np.sign(x) * np.exp(4.0 * np.abs(x))
    elif kind == "two":
        x = x * 1.0e-3
        x[n // 2:] += 100.0
    elif kind == "copies":                    # most points the same: the median is 0
        x[: 9 * n // 10] = 0.25
    elif kind == "levels":                    # a lattice beside a continuum
        x[: n // 2] = rng.integers(0, 2, size=(n // 2, 16))
    return torch.from_numpy(x.astype(np.float32)).cuda()


@pytest.mark.parametrize("kind", ["binary", "onehot", "halves", "outlier", "heavy", "two", "copies", "levels"])
@pytest.mark.parametrize("n", [37, 300, 512, 513, 1700, 5003])
def test_median_of_uneven_similarities(kind, n):
    S, p = apx.ap_similarity(_uneven(kind, n), noise_rel=0.0)
    assert p == _median(S)


@pytest.mark.parametrize("kind", ["binary", "onehot", "outlier", "heavy", "two"])
def test_uneven_similarities_do_not_cost_a_multiple(kind):
    """At 20000 points one-hot rows cost 5.2 times the plain points' build, two
    far clusters 3.4 times, when they went to the select over S."""
    n = 20000
    S = apx.empty_matrix(n)

    def best(X):
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            apx.ap_similarity(X, S, noise_rel=0.0)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    assert best(_uneven(kind, n)) < 2.5 * best(_uneven("plain", n))
