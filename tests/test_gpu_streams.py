"""GPU tests of one-launch steps of several workspaces on streams of the
caller's own: more work-groups than the compute units hold together."""
import time

import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu


def _workspaces(L, n, dtype):
    b = qk.qk_basis_build(L, L // 2)
    out = []
    for i in range(n):
        k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, True, random_fields(L, 40 + i)), 30, dtype)
        x = random_complex(qk.qk_basis_dim(b), 50 + i)
        out.append((k, x / np.linalg.norm(x)))
    return out


def _rounds(ws, psis, streams, n):
    """Milliseconds of n steps of every workspace, each on its own stream."""
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(n):
        for (k, _), psi, s in zip(ws, psis, streams):
            qk.qk_krylov_expm_step(k, psi, 0.05, stream=s)
    torch.cuda.synchronize()
    return 1e3 * (time.perf_counter() - t) / n


@pytest.mark.parametrize("L,n,dtype", [(19, 3, torch.complex128), (19, 3, torch.complex64), (20, 4, torch.complex128)])
def test_steps_that_do_not_fit_together(L, n, dtype):
    # they take their turns: the same bits as on one stream, and no slower than
    # half as long again (get a part of the device each and wait for the rest:
    # four to seven times as long)
    ws = _workspaces(L, n, dtype)
    streams = [torch.cuda.Stream() for _ in range(n)]
    times, states = {}, {}
    for name, on in (("one stream", streams[:1] * n), ("streams of their own", streams)):
        say(name, L, n, dtype)
        psis = [to_dev(x, dtype) for _, x in ws]
        _rounds(ws, psis, on, 3)
        times[name] = min(_rounds(ws, psis, on, 10) for _ in range(5))
        states[name] = [to_host(p) for p in psis]
    say(times)
    for a, b in zip(*states.values()):
        assert np.array_equal(a, b)
    assert times["streams of their own"] < 1.5 * times["one stream"]


def test_several_threads():
    # the order is kept under a lock: threads that step their own workspaces on
    # their own streams, and one that creates and destroys others meanwhile
    import threading
    L, n, steps, dtype = 19, 3, 40, torch.complex128
    ws = _workspaces(L, n, dtype)
    want = []
    for k, x in ws:
        psi = to_dev(x, dtype)
        for _ in range(steps):
            qk.qk_krylov_expm_step(k, psi, 0.05)
        want.append(to_host(psi))
    psis = [to_dev(x, dtype) for _, x in ws]
    streams = [torch.cuda.Stream() for _ in range(n + 1)]
    torch.cuda.synchronize()
    say("threads")

    def step(i):
        for _ in range(steps):
            qk.qk_krylov_expm_step(ws[i][0], psis[i], 0.05, stream=streams[i])

    def others():
        for _ in range(5):
            for k, x in _workspaces(16, 2, dtype):
                psi = to_dev(x, dtype)
                qk.qk_krylov_expm_step(k, psi, 0.05, stream=streams[n])

    threads = [threading.Thread(target=step, args=(i,)) for i in range(n)] + [threading.Thread(target=others)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for psi, w in zip(psis, want):
        assert np.array_equal(to_host(psi), w)
