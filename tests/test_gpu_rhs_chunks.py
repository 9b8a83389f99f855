"""The unfused right-hand side and its assembly at the sizes where their tiles
can go wrong: layer counts below, at and just past a workgroup's layers and
levels for every order (rows that end inside, at the end of and just past 16
levels; node counts off the assembly's 64), hanging columns, walls; against the
oracle (floor-scaled relative L2 <= 1e-12 per field, the bar of every FP64
call)."""

import numpy as np
import pytest

from oracle import assembly, metrics
from test_gpu_parity import TOL64, Setup, _element_contrib, _gpu_rhs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nz,periodic", [
    (1, 1, True), (1, 15, True), (1, 17, False), (2, 8, True), (2, 9, False), (3, 5, True), (3, 9, False),
    (4, 4, True), (4, 5, False), (5, 3, True), (6, 1, False), (6, 3, True), (7, 2, False), (8, 2, True)])
def test_rhs_and_assembly_match_oracle(N, nz, periodic):
    say("rhs chunks", N, nz, periodic)
    S = Setup("small_amr3", dict(N=N, periodic=periodic, z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1) ** 1.05))
    torch, api = S.torch, S.api
    hv = torch.zeros(S.gm.n_hstate, dtype=torch.float64, device="cuda")
    api.sem_nc_project(S.gm, api.SEM_SCATTER, S.q_g, hv)
    rE = torch.full((5 * S.gm.n_local,), float("nan"), dtype=torch.float64, device="cuda")
    api.sem_rhs(S.gm, S.q_g, hv, rE, api.SEM_FP64)
    torch.cuda.synchronize()
    err = metrics.rel_l2(rE.cpu().numpy().reshape(5, -1), _element_contrib(S), metrics.RHS_FLOORS * S.om.mL.mean())
    say("  rel elements", err)
    assert err.max() <= TOL64
    want = assembly.rhs(S.om, S.q_or, S.ref, S.c["phys"])
    err = metrics.rel_l2(S.to_oracle_order(_gpu_rhs(S, api.SEM_FP64)), want, metrics.RHS_FLOORS)
    say("  rel assembled", err)
    assert err.max() <= TOL64
