"""GPU test of the mixed ensemble -- 64 phases of the 20-site ring with single
rings of 16, 18, 20 and 22 sites -- against the oracle's stored survival
probabilities, by direct launches on several streams (no graph)."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_host
from test_gpu_batch import _golden_batch, _ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-10), (torch.complex64, 1e-5)])
def test_first_times_of_the_mixed_ensemble(dtype, tol):
    # the bounds are those of the run to t = 50
    times, members, Pref = _golden_batch()
    ws = [_ws(L, Bn, dtype, seed=i) for i, (L, Bn) in enumerate([(20, 64), (16, 1), (18, 1), (20, 1), (22, 1)])]
    assert [L for L, _ in members] == [20] * 64 + [16, 18, 20, 22] and list(times[:3]) == [1.0, 2.0, 3.0]
    bt = qk.qk_batch_create([w["k"] for w in ws], [w["psi"] for w in ws], [w["r0"] for w in ws])
    say("mixed ensemble, direct launches", dtype)
    P = to_host(qk.qk_batch_run(bt, 0.1, 30, use_graph=0))
    err = np.abs(P[[9, 19, 29]] - Pref[:3])
    say("max |dP| per time", err.max(axis=1))
    assert err.max() < tol
