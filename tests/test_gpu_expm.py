"""GPU tests of the projected exponential over the range of its argument, from
two terms to thousands, both signs, one and several vectors."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from oracle import hamiltonian as OH
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.mark.parametrize("L,N,m", [(2, 1, 2), (3, 1, 3), (6, 3, 20), (8, 2, 28), (7, 3, 35), (8, 3, 56)])
@pytest.mark.parametrize("dt", [0.0, 1e-23, 1e-21, 1e-12, 1e-3, 0.1, -0.1, 1.0, -7.0, 100.0, 2000.0])
def test_whole_subspace_vs_dense(L, N, m, dt):
    # a Krylov space of the sector's dimension, reorthogonalised: the step is the
    # exponential of the whole Hamiltonian up to rounding
    f = random_fields(L, 40 + L)
    b = qk.qk_basis_build(L, N)
    D = qk.qk_basis_dim(b)
    assert m == D
    H = OH.build_csr(L, N, False, 1.0, 0.7, f).toarray()
    lam, Q = np.linalg.eigh(H)
    k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, False, f), m, torch.complex128, reorth=2)
    x = random_complex(D, 8)
    x /= np.linalg.norm(x)
    psi = to_dev(x)
    say("whole subspace", L, N, m, dt)
    qk.qk_krylov_expm_step(k, psi, dt)
    ref = Q @ (np.exp(-1j * dt * lam) * (Q.T @ x))
    # eigenvalues of either side are off by at most a few roundings a row of the norm
    norm = np.max(np.abs(lam))
    assert np.linalg.norm(to_host(psi) - ref) < 8 * D * EPS * (1.0 + abs(dt) * norm)
