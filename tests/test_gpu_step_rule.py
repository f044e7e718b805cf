"""GPU test of the step-size rule of the adaptive evolution against the host:
the step it suggests after one whose error estimate lies below double
resolution, from the Lanczos coefficients and the rule's own series."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev
from oracle import model as OM
from workloads import BETA_GOLDEN, random_complex

pytestmark = pytest.mark.gpu


def _last_component(al, be, tau):
    """|exp(-i tau T) e_1| at its last row by the Taylor series in substeps of |tau| R
    <= 1/2 (T less the centre of its Gershgorin interval, R its radius), each
    ended by a term below 1e-18 of the sum."""
    left, right = np.r_[0.0, be], np.r_[be, 0.0]
    lo, hi = np.min(al - left - right), np.max(al + left + right)
    n = max(1, int(np.ceil(tau * 0.5 * (hi - lo) / 0.5)))
    v = np.zeros(len(al), complex)
    v[0] = 1.0
    size = lambda x: np.max(np.abs(x.real) + np.abs(x.imag))
    for _ in range(n):
        term = total = v
        for k in range(1, 41):
            term = -1j * (tau / n / k) * ((al - 0.5 * (lo + hi)) * term + left * np.r_[0.0, term[:-1]]
                                          + right * np.r_[term[1:], 0.0])
            total = total + term
            if size(term) <= 1e-18 * size(total):
                break
        v = total
    return abs(v[-1])


@pytest.mark.parametrize("passes", [False, True])
def test_suggested_step_below_double_resolution(passes):
    # the open 13-site chain: after a first step of 0.3 the estimate is about 1e-29 and
    # the suggestion 1.834; the exact component (7e-29, in a longer type) would move
    # it by 1.2e-5 of itself, a series summed in double to 1e-16 by half.  The
    # evolution takes 0.3, the suggestion, and the half of it that is left.
    L, m, tol, first = 13, 27, 1e-6, 0.3
    b = qk.qk_basis_build(L, 6)
    H = qk.qk_ham_create(b, 1.0, 1.0, False, OM.fields(L, 1.0, BETA_GOLDEN, 0.3))
    z = random_complex(qk.qk_basis_dim(b), 3)
    z /= np.linalg.norm(z)
    k = qk.qk_krylov_create(H, m)
    if passes:
        qk.qk_krylov_profile(k, True)   # kernel by kernel
    say("step rule, passes", passes)
    info = qk.qk_krylov_expm_step(k, to_dev(z), first, info=True)[0]
    al, be, used = qk.qk_krylov_coefficients(k)
    assert used == m
    err = info["beta0"] * be[m - 1] * _last_component(np.array(al[:m]), np.array(be[:m - 1]), first)
    assert 1e-30 < err < 1e-27
    want = 0.9 * first * (first * tol / err) ** (1.0 / (m - 1))
    got = qk.qk_krylov_evolve(k, to_dev(z), first + 1.5 * want, tol, dt_init=first)
    say(got, want)
    assert got["steps"] == 3 and got["dt_min"] == first
    # about a hundred roundings of the component, of which the suggestion has the 26th root
    assert abs(got["dt_max"] / want - 1) < 1e-13
