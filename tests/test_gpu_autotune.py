"""GPU tests of what the autotuner searches: nothing for workspaces whose step
takes one launch, distinct launches for the others."""
import json

import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu


def _workspace(L, Bn, dtype):
    b = qk.qk_basis_build(L, L // 2)
    hs = np.stack([random_fields(L, 20 + i) for i in range(Bn)])
    return qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, True, hs), 20, dtype)


def _step(k, dtype):
    D, Bn, _ = qk.qk_ham_shape(k.H)
    x = random_complex(D * Bn, 3).reshape(D, Bn)
    psi = to_dev(x / np.linalg.norm(x, axis=0), dtype)
    qk.qk_krylov_expm_step(k, psi, 0.05)
    return to_host(psi)


@pytest.mark.parametrize("L,Bn,dtype", [(16, 1, torch.complex64), (18, 4, torch.complex64), (20, 1, torch.complex64),
                                        (20, 1, torch.complex128)])
def test_a_step_in_one_launch_has_no_shape(tmp_path, L, Bn, dtype):
    say("autotune, one launch", L, Bn, dtype)
    k = _workspace(L, Bn, dtype)
    shape, want = qk.qk_krylov_get_shape(k), _step(k, dtype)
    cache = tmp_path / "tune.json"
    assert qk.qk_krylov_autotune(k, 0.05, cache) == shape
    assert qk.qk_krylov_get_shape(k) == shape
    assert np.array_equal(_step(k, dtype), want)
    # an entry that asks for other tiles is not taken
    (key, entry), = json.loads(cache.read_text()).items()
    entry.update(blocked_llo=max(entry["blocked_llo"] - 1, 0), threads=64, blocked_wgs_per_cu=4)
    cache.write_text("{\n  " + json.dumps(key) + ": " + json.dumps(entry) + "\n}\n")
    k2 = _workspace(L, Bn, dtype)
    assert qk.qk_krylov_autotune(k2, 0.05, cache) == shape
    assert np.array_equal(_step(k2, dtype), want)


@pytest.mark.parametrize("L,Bn,dtype", [(22, 1, torch.complex128), (21, 2, torch.complex64), (16, 16, torch.complex64)])
def test_work_groups_that_a_compute_unit_holds(L, Bn, dtype):
    # two or three fit; more was the same launch as all that fit, which is 0
    say("autotune, tiles", L, Bn, dtype)
    k = _workspace(L, Bn, dtype)
    assert qk.qk_krylov_autotune(k, 0.05)["blocked_wgs_per_cu"] in (0, 1, 2)
