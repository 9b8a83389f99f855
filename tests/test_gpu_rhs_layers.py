"""Every instance of the unfused right-hand side (layers per workgroup, picked by
the layer count), full and with empty layers, and both assemblies: as the tests
of its chunks, and in float at the bar of the float right-hand side (1e-4)."""

import pytest

import test_gpu_rhs_chunks as chunks
from oracle import metrics
from test_gpu_parity import Setup, _element_contrib, say

pytestmark = pytest.mark.gpu

LAYERS = {1: (2, 3, 6, 12, 16, 20), 2: (1, 2, 3, 4, 5), 3: (1, 2, 3, 4, 6, 7), 4: (1, 2, 3, 6, 8), 5: (1, 2)}


@pytest.mark.parametrize("N,nz", [(N, nz) for N in LAYERS for nz in LAYERS[N]])
def test_instances_match_oracle(N, nz):
    chunks.test_rhs_and_assembly_match_oracle(N, nz, True)


@pytest.mark.parametrize("N,nz", [(1, 5), (1, 9), (2, 3), (2, 6), (3, 3), (3, 4), (4, 2), (4, 5), (5, 3)])
def test_float_instances_match_oracle(N, nz):
    import numpy as np
    say("rhs layers, float", N, nz)
    S = Setup("small_amr3", dict(N=N, z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1) ** 1.05))
    hv = S.torch.zeros(S.gm.n_hstate, dtype=S.torch.float64, device="cuda")
    S.api.sem_nc_project(S.gm, S.api.SEM_SCATTER, S.q_g, hv)
    rE = S.torch.full((5 * S.gm.n_local,), float("nan"), dtype=S.torch.float64, device="cuda")
    S.api.sem_rhs(S.gm, S.q_g, hv, rE, S.api.SEM_FP32)
    S.torch.cuda.synchronize()
    err = metrics.rel_l2(rE.cpu().numpy().reshape(5, -1), _element_contrib(S), metrics.RHS_FLOORS * S.om.mL.mean())
    say("  rel elements", err)
    assert err.max() <= 1e-4
