"""GPU tests of the batched driver's graph: one workspace, its step captured
and replayed, against the same launches made directly -- forms whose step is
many launches, and records of any initial state."""
import numpy as np
import pytest
import torch

import paper_1704_02770_amd as qk
from gpu_util import say, to_dev, to_host
from workloads import random_complex, random_fields

pytestmark = pytest.mark.gpu

C128, C64 = torch.complex128, torch.complex64
# (L, N, phases, dtype, mode, reorth, use_graph)
CASES = [
    (22, 11, 1, C128, qk.QK_MATFREE, 0, 1), (22, 11, 1, C64, qk.QK_MATFREE, 0, 2),      # tiles
    (16, 8, 16, C64, qk.QK_MATFREE, 0, 1), (16, 8, 16, C128, qk.QK_MATFREE, 1, 2),      # totals of many columns
    (21, 10, 3, C128, qk.QK_MATFREE, 1, 1),                                             # no power of two
    (14, 7, 2, C128, qk.QK_MATFREE, 2, 1),                                              # full reorthogonalisation
    (14, 7, 3, C64, qk.QK_CSR, 0, 1), (15, 7, 1, C128, qk.QK_MATFREE_ROWS, 0, 2),       # rows
    (16, 8, 1, C128, qk.QK_MATFREE, 0, 1), (12, 6, 1, C64, qk.QK_MATFREE, 0, 2),        # one launch
]


@pytest.mark.parametrize("basis_state", [True, False])
@pytest.mark.parametrize("L,N,Bn,dtype,mode,reorth,use_graph", CASES)
def test_replays_equal_direct_launches(L, N, Bn, dtype, mode, reorth, use_graph, basis_state):
    hs = np.stack([random_fields(L, 60 + i) for i in range(Bn)])
    b = qk.qk_basis_build(L, N)
    k = qk.qk_krylov_create(qk.qk_ham_create(b, 1.0, 0.7, True, hs, mode), 12, dtype, reorth=reorth)
    x = random_complex(qk.qk_basis_dim(b) * Bn, 61).reshape(-1, Bn)
    x /= np.linalg.norm(x, axis=0)
    out = {}
    for g in (0, use_graph):
        say("batch of one workspace, mode", g, L, N, Bn, dtype, mode, reorth)
        psi = to_dev(x, dtype)
        bt = qk.qk_batch_create([k], [psi], [5 if basis_state else -1])
        P, C = (torch.empty((3, Bn), dtype=torch.float64, device="cuda") for _ in range(2))
        got = []
        for rep in range(3):
            qk.qk_batch_run_autocorr(bt, 0.05, 3, use_graph=g, out=P, out_c=C)
            got += [to_host(P).copy(), to_host(C).copy()]
            # eager work of the program between replays, and another step of the workspace
            assert np.isfinite(torch.randn(1000, device="cuda").sum().item())
            qk.qk_krylov_expm_step(k, to_dev(x, dtype), 0.02)
        out[g] = np.concatenate(got), to_host(psi)
    assert np.all(np.isfinite(out[0][0])) and np.any(out[0][1] != x.astype(out[0][1].dtype))
    for a, c in zip(out[0], out[use_graph]):
        assert np.array_equal(a, c)
