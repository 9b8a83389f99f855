"""The fused stage's owner kernel at the sizes where its chunks and roles can
go wrong: element counts below, at and just past whole chunks of every order
with an instance, walls, meshes one and two columns wide (a column beside
itself), two and three levels with hanging points, and pressures outside the
range of its polynomial, against the oracle (floor-scaled relative L2 <= 1e-12
per field, the bar of every FP64 call)."""

import numpy as np
import pytest

from oracle import assembly, metrics, timestep
from synth import columns
from test_gpu_parity import TOL64, Setup, say

pytestmark = pytest.mark.gpu


def _over(N, nx, ny, nz, periodic=True):
    return dict(N=N, nx0=nx, ny0=ny, Lx=4e5, Ly=3.5e5, columns=columns.uniform(nx, ny),
                z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1) ** 1.05, periodic_x=periodic, periodic_y=periodic)


CASES = {
    **{f"N{N}_nz{nz}": ("small_uniform", _over(N, 3, 2, nz))
       for N, L in [(2, 8), (3, 8), (4, 4), (5, 2), (6, 1), (7, 2), (8, 1)]
       for nz in sorted({1, max(1, L - 1), L, L + 1, 2 * L + 1})},
    **{f"N{N}_walls": ("small_uniform", _over(N, 3, 4, 5, periodic=False)) for N in range(2, 9)},
    "N4_one_wide": ("small_uniform", _over(4, 1, 3, 5)),
    "N5_one_column": ("small_uniform", _over(5, 1, 1, 3)),
    "N7_two_wide": ("small_uniform", _over(7, 2, 1, 3)),
    **{f"N{N}_amr3": ("small_amr3", dict(N=N)) for N in (2, 3, 5, 6, 8)},
    "N4_amr3_walls": ("small_amr3", dict(N=4, periodic=False)),
}


@pytest.mark.parametrize("far", [False, True], ids=["near", "far"])
@pytest.mark.parametrize("name", CASES)
def test_owner_stage_matches_oracle(name, far):
    case, kw = CASES[name]
    say("owner", name, far)
    S = Setup(case, kw)
    torch, api = S.torch, S.api
    q = S.q_or.copy()
    rng = np.random.default_rng(5)
    if far:
        # every eleventh node denser by 0.05 and warmer by 15 K: |(p / p0)^(1/gamma) - 1| > 1/64
        pick = rng.random(q.shape[1]) < 1 / 11
        q[0, pick] += 0.05
        q[4, pick] += 15.0
    qn = q * (1.0 + 1e-3 * rng.standard_normal(q.shape))
    dq, dqn = (S.gm.unpack(v[:, S.perm]) for v in (q, qn))
    R = assembly.rhs(S.om, q, S.ref, S.c["phys"])
    for st in (0, 1):
        a, b, c = timestep.stage_coefficients(st, S.c["dt"])
        out = torch.full_like(dq, float("nan"))
        api.sem_stage(S.gm, a, b, c, dqn, dq, out, api.SEM_FP64)
        torch.cuda.synchronize()
        want = timestep.stage_update(a, b, c, qn, q, R)
        err = metrics.rel_l2(S.to_oracle_order(out), want, metrics.STATE_FLOORS)
        say("  rel", err)
        assert err.max() <= TOL64
