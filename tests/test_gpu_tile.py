"""GPU tests of the tiled H x at the edges of its decomposition: the shortest
chains it takes, one particle and one hole, blocks of one row, batches on either
side of a power of two, chains whose tiles take several top patterns, and a
change of the fields after the tables are built."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import max_rel, say, to_dev, to_host
from oracle import basis as OB
from oracle import hamiltonian as OH
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu

# a row sums at most L + 1 products in either precision; the largest entry of H x
# is of the size of the largest row sum
EPS = {torch.complex128: 2.0 ** -52, torch.complex64: 2.0 ** -23}

CASES = [(7, 3, True, 1), (8, 4, True, 1), (8, 1, False, 1), (9, 8, True, 2), (10, 5, False, 3), (11, 4, True, 64),
         (12, 6, True, 33), (13, 6, False, 5), (14, 7, True, 1), (16, 2, True, 7), (17, 8, False, 8), (18, 9, True, 1),
         (19, 9, False, 2), (19, 17, True, 1), (21, 10, True, 1), (22, 11, False, 1)]


def _oracle(L, N, pbc, hs, X):
    H0 = OH.build_csr(L, N, pbc, 1.0, 0.7, np.zeros(L))
    st = OB.sector_states(L, N)
    dfield = OH.diagonal(st, L, pbc, 0.7, hs) - OH.diagonal(st, L, pbc, 0.7, np.zeros(L))[:, None]
    return H0 @ X + dfield * X


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("L,N,pbc,Bn", CASES)
def test_tiled_hv_vs_oracle(L, N, pbc, Bn, dtype):
    hs = np.stack([random_fields(L, 500 + i) for i in range(Bn)])
    b = qk.qk_basis_build(L, N)
    D = qk.qk_basis_dim(b)
    say("tiled hv", L, N, pbc, Bn, dtype)
    H = qk.qk_ham_create(b, 1.0, 0.7, pbc, random_fields(L, 1) + 0 * hs)
    x = to_dev(random_complex(D * Bn, 60 + L).reshape(D, Bn), dtype)
    qk.qk_ham_set_fields(H, hs)
    ref = _oracle(L, N, pbc, hs, to_host(x).astype(np.complex128))
    assert max_rel(to_host(qk.qk_ham_apply(H, x)), ref) < 4 * (L + 1) * EPS[dtype]


@pytest.mark.parametrize("L,N,Bn,reorth", [(8, 4, 1, 0), (12, 5, 3, 1), (18, 9, 1, 1), (18, 9, 2, 0), (19, 9, 1, 0)])
def test_tiled_steps_follow_the_row_form(L, N, Bn, reorth):
    # the H-pass with its sums, through the tables and one row per thread
    dtype = torch.complex64
    hs = np.stack([random_fields(L, 700 + i) for i in range(Bn)])
    b = qk.qk_basis_build(L, N)
    D = qk.qk_basis_dim(b)
    x = random_complex(D * Bn, 9).reshape(D, Bn)
    x /= np.linalg.norm(x, axis=0)
    out = []
    for mode in (qk.QK_MATFREE, qk.QK_MATFREE_ROWS):
        say("tiled steps", L, N, Bn, reorth, mode)
        k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, True, hs, mode), 16, dtype, reorth=reorth)
        psi = to_dev(x, dtype)
        for _ in range(3):
            qk.qk_krylov_expm_step(k, psi, 0.05)
        out.append(to_host(psi))
    # three steps of 16 vectors, each with a few roundings of every element
    assert np.max(np.abs(out[0] - out[1])) < 3 * 16 * 4 * EPS[dtype] * np.max(np.abs(out[1]))
