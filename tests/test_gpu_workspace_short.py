"""Calls on a device that has no memory left for the part of the workspace a
call can do without: a stand-in for hipMalloc, ahead of the runtime's in the
symbol search of a child process, refuses allocations above a limit.
"""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static int (*real)(void **, size_t);
static size_t most = ~(size_t)0;
void limit(const char *runtime, size_t bytes) {
    if (!real) real = (int (*)(void **, size_t))dlsym(dlopen(runtime, RTLD_LAZY | RTLD_NOLOAD), "hipMalloc");
    most = bytes;
}
int hipMalloc(void **p, size_t bytes) { return bytes > most ? 2 /* out of memory */ : real(p, bytes); }
"""

CHILD = r"""
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.limit.argtypes = [ctypes.c_char_p, ctypes.c_size_t]
sys.path.insert(0, sys.argv[2])
import torch
runtime = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
def limit(b): shim.limit(runtime.encode(), b)
limit(1 << 62)
import paper_0910_1650_amd as apx
"""


def _child(tmp_path, body):
    so = str(tmp_path / "shim.so")
    (tmp_path / "shim.c").write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", so, str(tmp_path / "shim.c"), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD + textwrap.dedent(body), so, ROOT], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "finished" in r.stdout, r.stdout + r.stderr


def test_median_without_memory_for_its_window(tmp_path):
    _child(tmp_path, """
        X = torch.randn(3000, 8, generator=torch.Generator().manual_seed(1)).cuda()
        few = 4 * 3000 + (1 << 18)
        S, S2 = apx.empty_matrix(3000), apx.empty_matrix(3000)
        limit(2 * few)
        S, p = apx.ap_similarity(X, S, noise_seed=3)
        assert apx.apx_workspace_bytes() <= 2 * few
        limit(1 << 62)
        S2, p2 = apx.ap_similarity(X, S2, noise_seed=3)
        assert apx.apx_workspace_bytes() >= apx.apx_workspace_size(apx.APX_OP_SIMILARITY, n=3000) > 2 * few
        assert p == p2 and torch.equal(S, S2)
        X, S = X[:1000], S[:1000, :1000]
        tiny = torch.empty(256, dtype=torch.uint8, device="cuda")
        apx.apx_set_workspace(tiny)
        apx.apx_set_workspace(None)
        limit(1 << 12)
        try:
            apx.ap_similarity(X, S)
        except apx.ApxError as e:
            assert e.status == apx.APX_ENOMEM
        else:
            raise SystemExit("no error")
        print("finished")
    """)


def test_landmarks_without_memory_for_the_window():
    import torch

    import paper_0910_1650_amd as apx

    X = torch.randn(2000, 4, generator=torch.Generator().manual_seed(2)).cuda()
    idx, res, ex = apx.lap_solve(X, 20, seed=4)
    # 20 landmarks: 4 MB of set-aside keys, a few hundred KB for everything else
    room = apx.apx_workspace_size(apx.APX_OP_LAP, n=2000, d=4, count=20) - (3 << 20)
    buf = torch.empty(room, dtype=torch.uint8, device="cuda")
    apx.apx_set_workspace(buf)
    try:
        idx2, res2, ex2 = apx.lap_solve(X, 20, seed=4)
    finally:
        apx.apx_set_workspace(None)
    assert torch.equal(idx, idx2) and res == res2 and list(ex) == list(ex2)
