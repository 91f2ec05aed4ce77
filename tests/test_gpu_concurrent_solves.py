"""Solves of several contexts, a host thread and a stream each: the launches
whose workgroups wait for each other share the device, and every result is
that of the call alone.
"""
import ctypes
import threading
import time

import pytest
import torch

import paper_0910_1650_amd as apx
import synth

pytestmark = pytest.mark.gpu

P = ctypes.c_void_p


def _s(n):
    pts = synth.gaussian_mixture(n=n, d=8, k=9, seed=n)
    return apx.ap_similarity(torch.from_numpy(pts.X).cuda(), noise_seed=n)[0]


class Caller:
    """A context on a stream of its own, and what its calls need."""

    def __init__(self, sizes):
        self.stream = torch.cuda.Stream()
        self.ctx = P()
        assert apx.lib().apx_create(ctypes.byref(self.ctx), torch.cuda.current_device(), P(self.stream.cuda_stream)) == 0
        self.S = [_s(n) for n in sizes]
        self.R, self.A = ([apx.empty_matrix(n) for n in sizes] for _ in "RA")
        self.idx = [torch.empty(n, dtype=torch.int32, device="cuda") for n in sizes]
        self.prm = apx.apx_params(0.9, 60, 15, 0, 0, 0.0)
        self.inst = (apx.apx_instance * len(sizes))(*[
            apx.apx_instance(n, S.stride(0), S.data_ptr(), R.data_ptr(), A.data_ptr(), i.data_ptr())
            for n, S, R, A, i in zip(sizes, self.S, self.R, self.A, self.idx)])
        self.res = (apx.apx_result * len(sizes))()

    def call(self):
        L, i = apx.lib(), self.inst[0]
        if len(self.inst) > 1:
            st = L.ap_solve_batched(self.ctx, len(self.inst), self.inst, 0, ctypes.byref(self.prm), self.res)
        else:
            st = L.ap_solve(self.ctx, i.S, i.n, i.ld, i.R, i.A, 0, ctypes.byref(self.prm), i.idx,
                            ctypes.byref(self.res[0]))
        assert st == 0, L.apx_last_error(self.ctx)

    def out(self):
        return [x.clone() for x in (*self.idx, *self.R, *self.A)]

    def close(self):
        apx.lib().apx_destroy(self.ctx)


def _together(callers, reps):
    fail = []

    def work(c):
        try:
            torch.cuda.set_device(0)
            for _ in range(reps):
                c.call()
        except BaseException as e:      # noqa: BLE001 (reported below)
            fail.append(e)

    threads = [threading.Thread(target=work, args=(c,)) for c in callers]
    t0 = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not fail, fail
    return time.perf_counter() - t0


@pytest.mark.parametrize("kinds", [
    [[300], [300], [300], [300]],
    [[60], [500], [1000], [2000], [3000], [700]],
    [[2400], [40, 300, 900], [3100, 200], [1500], [64] * 30, [2000, 2100]],
])
def test_results_are_those_of_a_call_alone(kinds):
    callers = [Caller(k) for k in kinds]
    torch.cuda.synchronize()
    alone = []
    for c in callers:
        c.call()
        alone.append(c.out())
        for m in (*c.R, *c.A):
            m.fill_(7.0)
    torch.cuda.synchronize()
    _together(callers, 12)
    for c, ref in zip(callers, alone):
        assert all(torch.equal(a, b) for a, b in zip(c.out(), ref))
        c.close()


def test_small_solves_share_the_device():
    """Four threads finish well before four times one thread's time (they took
    0.93 of it when the launches ran one after another)."""
    callers = [Caller([300]) for _ in range(4)]
    torch.cuda.synchronize()
    _together(callers, 5)
    one = min(_together(callers[:1], 60) for _ in range(3))
    four = min(_together(callers, 60) for _ in range(3))
    for c in callers:
        c.close()
    assert four < 0.65 * 4 * one
