"""GPU test of a decomposition that leaves more top bits than the tables hold
(31 sites with few particles, nine low bits in complex64): the rows are taken
one by one."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import max_rel, say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 4, 28])
def test_more_top_bits_than_the_tables_hold(N):
    L = 31
    say("21 top bits", L, N)
    h = random_fields(L, 8)
    b = qk.qk_basis_build(L, N)
    H, rows = qk.qk_ham_create(b, 1.0, 0.7, True, h), qk.qk_ham_create(b, 1.0, 0.7, True, h, qk.QK_MATFREE_ROWS)
    k = qk.qk_krylov_create(H, 12, torch.complex64)
    z = random_complex(qk.qk_basis_dim(b), 9)
    z /= np.linalg.norm(z)
    x, x2 = to_dev(z, torch.complex64), to_dev(z)
    default = to_host(qk.qk_ham_apply(H, x))
    want, want2 = to_host(qk.qk_ham_apply(rows, x)), to_host(qk.qk_ham_apply(rows, x2))
    qk.qk_krylov_set_shape(k, blocked_llo=9)
    assert np.array_equal(to_host(qk.qk_ham_apply(H, x)), want)   # the row form
    assert max_rel(to_host(qk.qk_ham_apply(H, x2)), want2) < 1e-14
    psi = to_dev(z, torch.complex64)
    qk.qk_krylov_expm_step(k, psi, 0.05)
    ref = to_dev(z)
    qk.qk_krylov_expm_step(qk.qk_krylov_create(rows, 12), ref, 0.05)
    assert max_rel(to_host(psi), to_host(ref)) < 1e-5
    qk.qk_krylov_set_shape(k, blocked_llo=11)
    assert np.array_equal(to_host(qk.qk_ham_apply(H, x)), default)
