"""The column kernel at N = 1, where a chunk's slice of the vertical tables (70
entries with eight layers) is longer than its nodes (36): every layers per
chunk and thread order, layer counts below, at and past a chunk, against the
oracle (FP64 1e-12 floor-scaled, the bar of every FP64 call; float 1e-4, that of
the float right-hand side)."""

import numpy as np
import pytest

from oracle import assembly, metrics, timestep
from test_gpu_parity import TOL64, Setup, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [1, 7, 8, 9, 17])
def test_stage_matches_oracle(nz):
    say("N = 1 stage", nz)
    S = Setup("small_amr3", dict(N=1, z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1) ** 1.05))
    torch, api = S.torch, S.api
    a, b, c = timestep.stage_coefficients(1, S.c["dt"])
    want = timestep.stage_update(a, b, c, S.q_or, S.q_or, assembly.rhs(S.om, S.q_or, S.ref, S.c["phys"]))
    for lpc in (1, 2, 4, 8):
        for layout in (0, 2, 3):
            if layout == 3 and lpc == 1:
                continue
            api.sem_stage_set_layout(S.gm, layout, lpc)
            for prec, tol in ((api.SEM_FP64, TOL64), (api.SEM_FP32, 1e-4)):
                out = torch.full_like(S.q_g, float("nan"))
                api.sem_stage(S.gm, a, b, c, S.q_g, S.q_g, out, prec)
                torch.cuda.synchronize()
                err = metrics.rel_l2(S.to_oracle_order(out), want, metrics.STATE_FLOORS)
                assert err.max() <= tol, (lpc, layout, prec, err)
