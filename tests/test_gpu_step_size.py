"""GPU test of the adaptive evolution's first steps, whose error estimates are
below the resolution of double precision: the step in one launch takes the same
steps as the passes do, and as a short first step is told to take."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,m", [(8, 4, 24), (13, 6, 27), (14, 7, 20), (16, 8, 12), (20, 10, 30)])
@pytest.mark.parametrize("dt_init", [1e-3, 0.1])
def test_one_launch_takes_the_steps_of_the_passes(L, N, m, dt_init):
    b = qk.qk_basis_build(L, N)
    D = qk.qk_basis_dim(b)
    H = qk.qk_ham_create(b, 1.0, 1.0, False, random_fields(L, 3))
    k = qk.qk_krylov_create(H, m, torch.complex128)
    x = random_complex(D, 4)
    x /= np.linalg.norm(x)
    out = []
    for profile in (False, True):
        say("step sizes", L, N, m, dt_init, profile)
        qk.qk_krylov_profile(k, profile)
        psi = to_dev(x)
        info = qk.qk_krylov_evolve(k, psi, 1.5, 1e-6, dt_init=dt_init)
        out.append((info, to_host(psi)))
    (a, pa), (c, pc) = out
    assert a["steps"] == c["steps"]
    # a step follows from an estimate to the power 1 / (m - 1); the coefficients
    # differ by roundings
    assert abs(a["dt_max"] - c["dt_max"]) < 1e-9 * c["dt_max"]
    assert np.max(np.abs(pa - pc)) < 1e-10
