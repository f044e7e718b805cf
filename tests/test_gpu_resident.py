"""GPU tests of the recurrence in one launch that small sectors take: one
work-group and many, rows that do not fill the last one, batches, the bond
counts at which its form changes, breakdowns, rows dealt out among few
work-groups, several workspaces on several streams, and graph replays."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu

EPS = {torch.complex128: 2.0 ** -52, torch.complex64: 2.0 ** -23}

# (L, N, ring, phases)
CASES = [(2, 1, False, 1), (5, 4, True, 3), (8, 4, True, 1), (11, 5, False, 1), (12, 6, True, 3), (14, 7, True, 1),
         (14, 7, True, 8), (15, 7, False, 5), (17, 8, True, 1), (18, 9, False, 1), (18, 2, True, 8), (19, 9, True, 2),
         (20, 10, True, 1)]


def _workspace(L, N, pbc, Bn, dtype, m, mode=qk.QK_MATFREE, reorth=0):
    hs = np.stack([random_fields(L, 900 + i) for i in range(Bn)])
    return qk.qk_krylov_create(qk.qk_ham_create(qk.qk_basis_build(L, N), 1.0, 0.7, pbc, hs, mode), m, dtype, reorth=reorth)


def _state(k, seed, dtype):
    D, Bn, _ = qk.qk_ham_shape(k.H)
    x = random_complex(D * Bn, seed).reshape(D, Bn)
    return to_dev(x / np.linalg.norm(x, axis=0), dtype)


def _steps(k, seed, dtype, n=2):
    psi = _state(k, seed, dtype)
    for _ in range(n):
        qk.qk_krylov_expm_step(k, psi, 0.05)
    return to_host(psi)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("L,N,pbc,Bn", CASES)
def test_one_launch_follows_the_passes(monkeypatch, L, N, pbc, Bn, dtype):
    m = 12
    say("resident", L, N, pbc, Bn, dtype)
    k = _workspace(L, N, pbc, Bn, dtype, m)
    one = _steps(k, 5, dtype)
    used = [qk.qk_krylov_coefficients(k, i)[2] for i in range(Bn)]
    qk.qk_krylov_profile(k, True)   # kernel by kernel
    passes = _steps(k, 5, dtype)
    assert used == [qk.qk_krylov_coefficients(k, i)[2] for i in range(Bn)]
    # two steps of m vectors, each with a few roundings of every element
    tol = 2 * m * 4 * EPS[dtype] * np.max(np.abs(passes))
    assert np.max(np.abs(one - passes)) < tol
    rows = _steps(_workspace(L, N, pbc, Bn, dtype, m, qk.QK_MATFREE_ROWS), 5, dtype)
    assert np.max(np.abs(one - rows)) < tol
    for n in ("1", "3"):   # few work-groups take all rows: the same sums in the same order
        say("resident, dealt out to", n)
        monkeypatch.setenv("QK_RESIDENT_JOIN", n)
        assert np.array_equal(_steps(_workspace(L, N, pbc, Bn, dtype, m), 5, dtype), one)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("L,N,pbc,Bn", [(8, 4, True, 1), (11, 5, False, 2), (13, 6, True, 1), (14, 7, False, 8),
                                        (16, 8, True, 3), (18, 9, True, 1), (19, 9, False, 1), (20, 10, True, 1)])
def test_local_reorthogonalisation_follows_the_passes(monkeypatch, L, N, pbc, Bn, dtype):
    m = 12
    say("resident reorth", L, N, pbc, Bn, dtype)
    k = _workspace(L, N, pbc, Bn, dtype, m, reorth=1)
    one = _steps(k, 5, dtype)
    plain = _steps(_workspace(L, N, pbc, Bn, dtype, m), 5, dtype)
    qk.qk_krylov_profile(k, True)   # kernel by kernel
    passes = _steps(k, 5, dtype)
    # as above, and one more product and sum of every element
    tol = 2 * m * 5 * EPS[dtype] * np.max(np.abs(passes))
    assert np.max(np.abs(one - passes)) < tol
    assert not np.array_equal(one, plain)   # it does something
    say("resident reorth, dealt out")
    monkeypatch.setenv("QK_RESIDENT_JOIN", "2")
    assert np.array_equal(_steps(_workspace(L, N, pbc, Bn, dtype, m, reorth=1), 5, dtype), one)


def test_columns_that_end_early():
    # column 0 zero, column 1 an eigenvector (all spins but one up: H acts on the
    # D = L one-magnon states), column 2 general: each stops on its own
    L, m, dtype = 14, 10, torch.complex128
    k = qk.qk_krylov_create(qk.qk_ham_create(qk.qk_basis_build(L, 1), 1.0, 0.7, True, np.zeros((3, L))), m, dtype)
    x = np.zeros((L, 3), np.complex128)
    x[:, 1] = 1.0 / np.sqrt(L)
    x[:, 2] = random_complex(L, 3)
    psi = to_dev(x, dtype)
    say("resident columns")
    used = [i["m_used"] for i in qk.qk_krylov_expm_step(k, psi, 0.1, info=True)]
    assert used[:2] == [0, 1] and used[2] > 5, used
    out = to_host(psi)
    assert np.all(out[:, 0] == 0)
    assert abs(np.linalg.norm(out[:, 1]) - 1) < 1e-13
    assert abs(np.linalg.norm(out[:, 2]) - np.linalg.norm(x[:, 2])) < 1e-12


def test_workspaces_on_many_streams():
    # more work-groups than the chip holds at once: whoever is late leaves its
    # rows to the others, with the same bits
    dtype = torch.complex128
    specs = [(16, 8, True, 1), (18, 9, False, 1), (14, 7, True, 8), (17, 8, True, 2), (19, 9, False, 1), (12, 6, True, 1)]
    ks = [_workspace(*s, dtype, 16) for s in specs]
    say("resident streams")
    want = [_steps(k, 7, dtype, 4) for k in ks]
    streams = [torch.cuda.Stream() for _ in ks]
    psi = [_state(k, 7, dtype) for k in ks]
    torch.cuda.synchronize()
    for _ in range(4):
        for k, p, s in zip(ks, psi, streams):
            with torch.cuda.stream(s):
                qk.qk_krylov_expm_step(k, p, 0.05, stream=s)
    torch.cuda.synchronize()
    for w, p in zip(want, psi):
        assert np.array_equal(to_host(p), w)


def test_graph_replays():
    L, dtype, steps = 16, torch.complex128, 6
    k = _workspace(L, L // 2, True, 2, dtype, 12)
    want = to_host(_state(k, 11, dtype))
    x = _state(k, 11, dtype)
    other = _workspace(15, 7, True, 1, dtype, 12)
    kept = _steps(other, 2, dtype)
    say("resident graph")
    outs = []
    for graph in (True, False):
        psi = x.clone()
        b = qk.qk_batch_create([k], [psi], [0])
        for _ in range(3):   # each call replays, with other work between
            qk.qk_batch_run(b, 0.05, steps, use_graph=graph)
            assert np.array_equal(_steps(other, 2, dtype), kept)
            torch.cuda.synchronize()
        outs.append(to_host(psi))
    assert np.array_equal(outs[0], outs[1]) and not np.array_equal(outs[0], want)
