"""What follows when workgroups of the one-launch solves give up waiting for
each other, forced from the host (every kernel still ends by itself): the
launched passes, or a batch's streaming launch, run from the caller's start.
"""
import numpy as np
import pytest
import torch

import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore():
    yield
    apx.apx_set_give_up(-1)
    apx.apx_set_graphs(True)


def _s(n):
    pts = synth.gaussian_mixture(n=n, d=8, k=9, seed=n)
    return apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=n)[0]


def _start(n, warm):
    g = torch.Generator().manual_seed(n)
    A = -torch.rand(n, n, generator=g)
    if warm == apx.APX_WARM_COLUMNS:
        A = -torch.rand(1, n, generator=g).repeat(n, 1)
    A.diagonal().abs_()
    return apx.to_matrix(torch.randn(n, n, generator=g)), apx.to_matrix(A)


KW = dict(damping=0.8, max_iter=60, conv_iter=15)


@pytest.mark.parametrize("warm", [apx.APX_COLD, apx.APX_WARM_A, apx.APX_WARM_AR, apx.APX_WARM_COLUMNS])
@pytest.mark.parametrize("n", [130, 700, 2400])
def test_a_solve_goes_on_in_the_launched_passes(n, warm):
    S = _s(n)
    out = []
    for graphs, at in ((False, -1), (True, 0), (True, 1), (True, 7)):
        apx.apx_set_graphs(graphs)
        apx.apx_set_give_up(at)
        R, A = _start(n, warm)
        idx, res = apx.ap_solve(S, R, A, warm=warm, **KW)
        assert apx.apx_last_fallback() == (apx.APX_FALLBACK_WAIT if graphs else 0)
        out.append((idx, R, A, res))
    for idx, R, A, res in out[1:]:
        assert torch.equal(idx, out[0][0]) and torch.equal(R, out[0][1]) and torch.equal(A, out[0][2])
        assert res == out[0][3]
    apx.apx_set_give_up(-1)
    apx.ap_solve(S, *_start(n, warm), warm=warm, **KW)
    assert apx.apx_last_fallback() == 0


def test_after_the_messages_are_written():
    n = 700
    S = _s(n)
    R, A = _start(n, apx.APX_COLD)
    ref, one = apx.ap_solve(S, R, A, **KW)
    apx.apx_set_give_up(-2)
    idx, res = apx.ap_solve(S, R, A, **KW)
    assert torch.equal(idx, ref) and res == one and apx.apx_last_fallback() == apx.APX_FALLBACK_WAIT
    for warm in (apx.APX_WARM_A, apx.APX_WARM_AR):
        with pytest.raises(apx.ApxError) as e:
            apx.ap_solve(S, *_start(n, warm), warm=warm, **KW)
        assert e.value.status == apx.APX_EDEVICE
    idx, res = apx.ap_solve(S[:5, :5], R[:5, :5], A[:5, :5], **KW)       # one workgroup waits for nothing
    assert apx.apx_last_fallback() == 0


@pytest.mark.parametrize("warm", [apx.APX_COLD, apx.APX_WARM_AR])
@pytest.mark.parametrize("at", [0, 1, 4])
def test_a_batch_goes_on_in_the_streaming_launch(at, warm, monkeypatch):
    sizes = [90, 400, 1100, 2500, 77, 640]
    Ss = [_s(n) for n in sizes]

    def run():
        RA = [_start(n, warm) for n in sizes]
        idxs, res = apx.ap_solve_batched(Ss, [r for r, _ in RA], [a for _, a in RA], warm=warm, **KW)
        return idxs, RA, res

    apx.apx_set_give_up(at)
    got = run()
    assert apx.apx_last_fallback() == apx.APX_FALLBACK_WAIT
    apx.apx_set_give_up(-1)
    run()
    assert apx.apx_last_fallback() == 0
    monkeypatch.setenv("APX_BATCH_WPC", "4")
    ref = run()
    for j in range(len(sizes)):
        assert torch.equal(got[0][j], ref[0][j]) and got[2][j] == ref[2][j]
        assert torch.equal(got[1][j][0], ref[1][j][0]) and torch.equal(got[1][j][1], ref[1][j][1])


def test_a_batch_after_the_messages_are_written():
    sizes = [90, 400]
    Ss = [_s(n) for n in sizes]
    ref, _ = apx.ap_solve_batched(Ss, **KW)
    apx.apx_set_give_up(-2)
    idxs, _ = apx.ap_solve_batched(Ss, **KW)
    for a, b in zip(idxs, ref):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    RA = [_start(n, apx.APX_WARM_AR) for n in sizes]
    with pytest.raises(apx.ApxError) as e:
        apx.ap_solve_batched(Ss, [r for r, _ in RA], [a for _, a in RA], warm=apx.APX_WARM_AR, **KW)
    assert e.value.status == apx.APX_EDEVICE
