"""GPU tests of the totals of the passes' partial sums: batches and block sizes
on either side of each branch of the reduction (whole waves with a power of two
of columns up to 32, any other column count, fewer threads than a wave)."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_host
from oracle import exact as OX
from oracle import hamiltonian as OH
from oracle import model as OM
from workloads import BETA_GOLDEN, phases, random_complex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bn,threads", [(1, 0), (1, 32), (2, 0), (2, 8), (3, 0), (3, 12), (5, 0), (7, 0), (8, 0),
                                        (32, 0), (33, 0), (64, 0), (64, 64)])
@pytest.mark.parametrize("reorth", [0, 1])
def test_step_of_every_reduction_shape(Bn, threads, reorth):
    L, dt, m = 10, 0.1, 20
    b = qk.qk_basis_build(L, L // 2)
    D = qk.qk_basis_dim(b)
    hf = np.stack([OM.fields(L, 1.5, BETA_GOLDEN, p) for p in phases(Bn, 3)])
    k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 1.0, True, hf), m, reorth=reorth)
    if threads:
        qk.qk_krylov_set_shape(k, threads=threads)
    x = random_complex(D * Bn, 5).reshape(D, Bn)
    x /= np.linalg.norm(x, axis=0)
    psi = torch.from_numpy(np.ascontiguousarray(x if Bn > 1 else x[:, 0])).to("cuda")
    say("reduction", Bn, threads, reorth)
    qk.qk_krylov_expm_step(k, psi, dt)
    got = to_host(psi).reshape(D, Bn)
    for c in range(Bn):
        Hd = OH.build_dense(L, L // 2, True, 1.0, 1.0, hf[c])
        ref = OX.evolve(Hd, x[:, c], np.array([dt]))[0]
        # m = 20 at dt |H| ~ 1 leaves the Krylov error below rounding: m eps times a few
        assert np.max(np.abs(got[:, c] - ref)) < 1e-12
