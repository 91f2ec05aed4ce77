"""The network's kernels at the edges of their tiles (32 points to a workgroup,
at most 256 workgroups with gradients, two per compute unit forward): one
point, around one tile and two, one more tile than workgroups, several tiles
per workgroup.  Tolerance of the gradients: one activation on the other side
of a bfloat16 rounding boundary (2^-8 of an entry), against each tensor's
largest; the forward pass as in its other tests (99% within 1e-4 of the output
scale, all within 2^-6).
"""
import numpy as np
import pytest
import torch

import paper_0910_1650_amd as apx
import synth
from oracle import warm

pytestmark = pytest.mark.gpu


def t32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("count", [1, 31, 32, 33, 64, 8192, 8193, 20011])
def test_gradient_tiles(count):
    theta = synth.mlp_params(3)
    X, T, w = synth.mlp_batch(count, 100 + count)
    g, loss = apx.apx_mlp_backward(t32(theta), t32(X), t32(T), t32(w))
    L, ref, _ = warm.backward(*(a.astype(np.float64) for a in (theta, X, T, w)), bf16=True)
    assert abs(loss.item() - L) <= 1e-5 * abs(L) + 2.0 ** -8 * abs(L) / count
    g = g.cpu().numpy().astype(np.float64)
    at = 0
    for name, shape in warm.SHAPES:
        size = int(np.prod(shape))
        a, b = g[at:at + size], ref[at:at + size]
        assert np.max(np.abs(a - b)) <= 2.0 ** -8 * np.max(np.abs(b)), name
        at += size


@pytest.mark.parametrize("count", [1, 33, 16384, 16385, 40001])
def test_forward_tiles(count):
    theta = synth.mlp_params(4)
    X, _, _ = synth.mlp_batch(count, 200 + count)
    y = apx.apx_mlp_forward(t32(theta), t32(X)).cpu().numpy().astype(np.float64)
    ref, c = warm.forward(theta.astype(np.float64), X.astype(np.float64), bf16=True)
    scale = np.max(np.abs(c["h2"]) @ np.abs(c["W3"]))
    err = np.abs(y - ref)
    assert np.all(err <= 2.0 ** -6 * scale)
    assert np.mean(err <= 1e-4 * scale) >= (0.99 if count > 100 else 0.9)


@pytest.mark.parametrize("count", [8192, 8224, 65536, 131072, 131136, 400000])
def test_partial_sums_stay_short(count):
    """The gradient of `count` copies of one row against `count` times that
    row's: equal addends, so FP32 sums over L of them differ from the product
    by at most (L + 1) 2^-24 of it.  L is at most 64 whatever the batch (the
    partials are added in FP64), plus one rounding of the result."""
    theta = t32(synth.mlp_params(5))
    X, T, w = (t32(a) for a in synth.mlp_batch(4, 5))
    one, l1 = apx.apx_mlp_backward(theta, X, T, w, rows=torch.full((1,), 2, device="cuda"))
    g, loss = apx.apx_mlp_backward(theta, X, T, w, rows=torch.full((count,), 2, device="cuda"))
    ref = one.double() * count
    assert bool(((g.double() - ref).abs() <= 66 * 2.0 ** -24 * ref.abs()).all())
    assert abs(loss.item() - count * l1.item()) <= 1e-12 * count * l1.item()
