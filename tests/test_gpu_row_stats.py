"""Row statistics of the warm-start features at the edges of their kernel: the
rows held in registers (up to 2, 4, 8, 16 elements per thread) and reread
above, rows whose values crowd into few intervals (ties, one far outlier, all
equal, both zeros) and so are cut again, next to rows that do not.
Order statistics are exact, so every feature equals the oracle's bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_0910_1650_amd as apx
import synth
from oracle import warm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 33, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193])
def test_features_equal_oracle(n):
    pts = synth.gaussian_mixture(n=n, d=8, k=5, seed=n)
    S, _ = apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=1)
    g = torch.Generator().manual_seed(n)
    if n > 100:
        S[1] = -3.0                                            # all equal
        S[2] = torch.randint(-4, 0, (n,), generator=g).float().cuda()   # four values
        S[3, 17] = -1.0e30                                     # one outlier: the rest in one interval
        S[4] = torch.where(torch.rand(n, generator=g) < 0.5, 0.0, -0.0).cuda()
        S[5] = -torch.arange(n).float().cuda()                 # evenly spread
    F, sig = apx.apx_features(S)
    rows = np.unique(np.concatenate([np.arange(min(n, 8)), np.random.default_rng(n).integers(0, n, 12)]))
    ref, _ = warm.features(S.cpu().numpy().astype(np.float64), rows=rows, sigma=float(sig))
    np.testing.assert_array_equal(F.cpu().numpy()[rows], ref.astype(np.float32))
    med = np.sort(np.partition(S.cpu().numpy()[~np.eye(n, dtype=bool)].reshape(n, n - 1), (n - 2) // 2, axis=1)[:, (n - 2) // 2])
    assert float(sig) == abs(med[(n - 1) // 2])


@pytest.mark.parametrize("n", [40, 700, 1500, 9000])
def test_values_that_are_not_finite(n):
    """Order statistics by the FP32 values' order with infinities at its ends
    and NaN above them (as numpy sorts)."""
    pts = synth.gaussian_mixture(n=n, d=8, k=5, seed=n)
    S, _ = apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=1)
    g = torch.Generator().manual_seed(n)
    S[1, 5] = float("nan")
    S[2, torch.randperm(n, generator=g)[:n // 3].cuda()] = float("nan")
    S[3, 7:9] = -float("inf")
    S[4, 7] = float("inf")
    S[5, ::2] = -float("inf")
    S[6, 9], S[6, 11], S[6, 12] = float("nan"), float("inf"), -float("inf")
    S[7, 8], S[7, 9] = -3.0e38, 3.0e38
    F, sig = apx.apx_features(S)
    M, m = S.cpu().numpy(), n - 1
    pos = [m - 1 - min(j, m - 1) for j in (0, 1, 3, 7, 15, 31)] + [q * (m - 1) // 100 for q in (1, 10, 25, 50, 75)]
    for k in range(9):
        row = np.sort(np.delete(M[k], k))
        with np.errstate(invalid="ignore"):
            ref = (row[pos].astype(np.float64) / float(sig)).astype(np.float32)
        np.testing.assert_array_equal(F.cpu().numpy()[k, [0, 1, 2, 3, 4, 5, 7, 8, 9, 10, 11]], ref)


@pytest.mark.parametrize("n", [66, 67, 258, 259, 700, 1026, 2048, 2049, 2300, 5000, 8192, 8193])
def test_rows_that_crowd(n):
    """Rows that take one to five cuts, beside each other in one call: ties at
    the ranks and between them, clusters inside clusters (each 2^-7 of the one
    around it), as many keys in one interval as a list may hold and one more."""
    pts = synth.gaussian_mixture(n=n, d=4, k=5, seed=n)
    S, _ = apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=1)
    rng = np.random.default_rng(n)
    rows = [np.full(n, -2.5), np.where(rng.random(n) < 0.5, -1.0, -2.0), -rng.integers(1, 6, n).astype(float)]
    for level in range(1, 6):
        r = -1.0 - rng.random(n)
        for j in range(1, level + 1):
            r[rng.permutation(n)[:n // (j + 1)]] = -1.5 - rng.random(n // (j + 1)) * 2.0 ** (-7 * j)
        rows.append(r)
    for held in (63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025):
        r = -1.0e6 * (1.0 + rng.random(n))
        r[:min(held, n)] = -rng.random(min(held, n))
        rows.append(rng.permutation(r))
    rows.append(-np.exp(rng.normal(0.0, 20.0, n)))
    rows.append(np.where(rng.random(n) < 0.9, -1.0, -rng.random(n)))
    rows.append(np.where(np.arange(n) < n - 3, -1.0e-38 * rng.integers(0, 4, n), -3.0e38))
    S[:len(rows)] = torch.from_numpy(np.stack(rows).astype(np.float32)).cuda()
    F, sig = apx.apx_features(S)
    ref, _ = warm.features(S.cpu().numpy().astype(np.float64), rows=np.arange(len(rows) + 2), sigma=float(sig))
    np.testing.assert_array_equal(F.cpu().numpy()[:len(rows) + 2], ref.astype(np.float32))


@pytest.mark.parametrize("n", [1000, 5000])
def test_an_outlier_does_not_cost_a_multiple(n):
    """One point far out puts all other values of every row into one interval
    (it cost 68 times the plain call at 1000 points)."""
    X = torch.randn(n, 16, generator=torch.Generator().manual_seed(3))

    def best(X):
        S, _ = apx.ap_similarity(X.cuda())
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                apx.apx_features(S)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    plain = best(X)
    X[0] = 1.0e4
    assert best(X) < 10 * plain
