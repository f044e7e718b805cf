"""GPU tests of a wait between the work-groups of a one-launch step that gives
up (QK_RESIDENT_POLLS, a limit set from the host: every work-group ends as
usual): the caller of every entry point learns of it, and psi is either the
step's result or what it was."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu

ENUMERIC = 5
# (L, N, ring, phases, dtype, reorth): forms with and without the exponential and the combination in the launch
CASES = [(16, 8, True, 1, torch.complex128, 0), (14, 7, False, 3, torch.complex64, 1), (20, 10, True, 1, torch.complex128, 0),
         (18, 9, False, 1, torch.complex64, 0)]


def _workspace(L, N, pbc, Bn, dtype, reorth, m=10):
    hs = np.stack([random_fields(L, 700 + i) for i in range(Bn)])
    b = qk.qk_basis_build(L, N)
    k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, pbc, hs), m, dtype, reorth=reorth)
    x = random_complex(qk.qk_basis_dim(b) * Bn, 11).reshape(-1, Bn)
    return k, to_dev(x / np.linalg.norm(x, axis=0), dtype)


@pytest.mark.parametrize("L,N,pbc,Bn,dtype,reorth", CASES)
def test_every_caller_learns_of_it(monkeypatch, L, N, pbc, Bn, dtype, reorth):
    say("gave up at once", L, N, pbc, Bn, dtype, reorth)
    monkeypatch.setenv("QK_RESIDENT_POLLS", "0")
    k, psi = _workspace(L, N, pbc, Bn, dtype, reorth)
    start = to_host(psi).copy()
    for _ in range(2):   # and the next step
        info = qk.qk_krylov_expm_step(k, psi, 0.05, info=True)
        assert [i["status"] for i in info] == [ENUMERIC] * Bn
        assert np.array_equal(to_host(psi), start)
    k, psi = _workspace(L, N, pbc, Bn, dtype, reorth)
    with pytest.raises(qk.QkError, match="gave up"):
        qk.qk_krylov_evolve(k, psi, 0.3, 1e-7, dt_init=0.1)
    assert np.array_equal(to_host(psi), start)
    for r0 in (3, -1):
        for graph in (0, 1):
            k, psi = _workspace(L, N, pbc, Bn, dtype, reorth)
            bt = qk.qk_batch_create([k], [psi], [r0])
            P, C = qk.qk_batch_run_autocorr(bt, 0.05, 3, use_graph=graph)
            assert np.all(np.isnan(to_host(P))) and np.all(np.isnan(to_host(C)))
            assert np.array_equal(to_host(psi), start)
    if Bn == 1 and dtype == torch.complex128:
        for keep in ("1", "0"):
            monkeypatch.setenv("QK_GRAD_KEEP", keep)
            k, _ = _workspace(L, N, pbc, Bn, dtype, reorth)
            with pytest.raises(qk.QkError, match="gave up"):
                qk.qk_grad_return_prob(k, 3, 0.2, 4)


@pytest.mark.parametrize("join", [None, "3"])
@pytest.mark.parametrize("L,N,pbc,Bn,dtype,reorth", CASES)
def test_the_result_or_nothing(monkeypatch, join, L, N, pbc, Bn, dtype, reorth):
    steps = 4
    k, psi = _workspace(L, N, pbc, Bn, dtype, reorth)
    states = [to_host(psi).copy()]
    for _ in range(steps):
        qk.qk_krylov_expm_step(k, psi, 0.05)
        states.append(to_host(psi).copy())
    if join:
        monkeypatch.setenv("QK_RESIDENT_JOIN", join)
    done = []
    for polls in (1, 2, 4, 8, 16, 32, 64, 128, 1000000):
        say("polls", polls, "join", join, L, N, pbc, Bn, dtype, reorth)
        monkeypatch.setenv("QK_RESIDENT_POLLS", str(polls))
        k, psi = _workspace(L, N, pbc, Bn, dtype, reorth)
        ok = []
        for _ in range(steps):
            info = qk.qk_krylov_expm_step(k, psi, 0.05, info=True)
            assert len({i["status"] for i in info}) == 1
            ok.append(info[0]["status"] == 0)
            assert np.array_equal(to_host(psi), states[sum(ok)])
        assert ok == sorted(ok, reverse=True)   # none succeeds after one that gave up
        done.append(sum(ok))
    say("steps that went through", done)
    assert done[-1] == steps
