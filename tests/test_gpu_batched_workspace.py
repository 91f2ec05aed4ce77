"""Batches of small and large instances on a caller's workspace: one of the
reported size serves the call, one that is too small leaves every output as it
was (also those of the instances that would have fitted).
"""
import pytest
import torch

import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu


def _batch():
    # one large instance among many of two points: alone it gets a larger team
    # (and more column partials) than beside them
    pts = synth.gaussian_mixture(n=4000, d=8, k=6, seed=5)
    big = apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=5)[0]
    pair = torch.tensor([[-0.5, -1.0], [-1.5, -0.25]])
    # (leading dimensions of a multiple of four, as the size query takes them)
    small = [torch.empty(2, 4, device="cuda")[:, :2] for _ in range(900)]
    for j, s in enumerate(small):
        s.copy_(pair - 0.01 * j)
    tight = torch.empty(4000, 4000, device="cuda")
    tight.copy_(big)
    return [tight, *small]


def test_the_reported_workspace_serves_a_mixed_batch():
    Ss = _batch()
    sizes = [S.shape[0] for S in Ss]

    def messages():
        return [torch.zeros(S.shape[0], S.stride(0), device="cuda")[:, :S.shape[0]] for S in Ss]

    R0, A0 = messages(), messages()
    ref, res = apx.ap_solve_batched(Ss, R0, A0, damping=0.9, max_iter=40, conv_iter=15)
    need = apx.apx_workspace_size(apx.APX_OP_SOLVE_BATCHED, count=len(sizes), sizes=sizes)
    buf = torch.empty(need, dtype=torch.uint8, device="cuda")
    apx.apx_set_workspace(buf)
    try:
        R, A = messages(), messages()
        idx, out = apx.ap_solve_batched(Ss, R, A, damping=0.9, max_iter=40, conv_iter=15)
    finally:
        apx.apx_set_workspace(None)
    assert out == res
    assert all(torch.equal(a, b) for x, y in ((idx, ref), (R, R0), (A, A0)) for a, b in zip(x, y))
    # room for the small instances' launch only
    few = apx.apx_workspace_size(apx.APX_OP_SOLVE_BATCHED, count=900, sizes=sizes[1:])
    buf = torch.empty(4 * few, dtype=torch.uint8, device="cuda")
    apx.apx_set_workspace(buf)
    try:
        R, A = messages(), messages()
        with pytest.raises(apx.ApxError) as e:
            apx.ap_solve_batched(Ss, R, A, damping=0.9, max_iter=40, conv_iter=15)
        assert e.value.status == apx.APX_ENOMEM
    finally:
        apx.apx_set_workspace(None)
    assert all(bool((m == 0).all()) for m in (*R, *A))
