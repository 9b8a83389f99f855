"""Both sides of the owner kernel's limits: 512 levels (its level table in LDS),
2 GiB of state (32-bit offsets), 768 columns at N = 7 (512 of one layer), the
columns up to which it pays for side columns.  Below, a default stage
runs it (reported layout (0, 0)); above, the coloured launches, to the bit of
those named.  Against the oracle at the bar of every FP64 call, or against the
named launches where the oracle would not fit."""

import numpy as np
import pytest

from oracle import assembly, gll, metrics, timestep
from synth import columns
from test_gpu_parity import TOL64, Setup, say

pytestmark = pytest.mark.gpu


def _kw(N, nx, ny, nz):
    return dict(N=N, nx0=nx, ny0=ny, Lx=4e5, Ly=3.5e5, columns=columns.uniform(nx, ny),
                z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1))


@pytest.mark.parametrize("N,nz", [(2, 255), (2, 256), (4, 127), (4, 128), (7, 73), (7, 74), (8, 63), (8, 64)])
def test_levels(N, nz):
    """At and just above 512 levels."""
    nzn = N * nz + 1
    say("levels", N, nzn)
    S = Setup("small_uniform", _kw(N, 3, 2, nz))
    torch, api = S.torch, S.api
    assert S.gm.info["nzn"] == nzn and (api.sem_stage_get_layout(S.gm) == (0, 0)) == (nzn <= 512)
    x = gll.lgl_nodes(N)
    dt = 0.4 * 0.5 * float(x[1] - x[0]) * 20e3 / nz / 390.0
    a, b, c = timestep.stage_coefficients(1, dt)
    out = torch.full_like(S.q_g, float("nan"))
    api.sem_stage(S.gm, a, b, c, S.q_g, S.q_g, out, api.SEM_FP64)
    torch.cuda.synchronize()
    want = timestep.stage_update(a, b, c, S.q_or, S.q_or, assembly.rhs(S.om, S.q_or, S.ref, S.c["phys"]))
    err = metrics.rel_l2(S.to_oracle_order(out), want, metrics.STATE_FLOORS)
    say("  rel", err)
    assert err.max() <= TOL64
    # the tendency alone: dp'/dz over layers a hundredth as deep as those of the
    # other tests, whose bar is 1e-12
    api.sem_stage(S.gm, 0.0, 0.0, 1.0, S.q_g, S.q_g, out, api.SEM_FP64)
    torch.cuda.synchronize()
    err = metrics.rel_l2(S.to_oracle_order(out), assembly.rhs(S.om, S.q_or, S.ref, S.c["phys"]), metrics.RHS_FLOORS)
    say("  rhs rel", err)
    assert err.max() <= 1e-10


def _against_named(N, nx, ny, nz, owner, periodic=True, **over):
    import torch
    from paper_2410_21607_amd import api
    say("limit", N, nx, ny, nz, owner)
    gm = api.Mesh.from_case(dict(_kw(N, nx, ny, nz), periodic_x=periodic, periodic_y=periodic,
                                 phys=dict(f=5e-5, g=9.81, R_d=287.0, c_p=1004.0, p00=1.0e5), **over))
    z = gm.coords()[2]
    gm.set_reference(1.2 * np.exp(-z / 8e3), 300.0 * np.exp(1e-5 * z), 3e-3 * np.exp(1e-5 * z))
    q = gm.state().view(5, -1, gm.ldz)
    g = torch.Generator(device="cuda").manual_seed(3)
    for f in range(5):
        q[f, :, :z.size] = 1e-3 * torch.randn(q[f, :, :z.size].shape, generator=g, dtype=torch.float64, device="cuda")
    q[0, :, :z.size] *= torch.as_tensor(np.exp(-z / 8e3), device="cuda")
    q = q.reshape(-1)
    assert (api.sem_stage_get_layout(gm) == (0, 0)) == owner
    outs = []
    for layout in (None, (0, api.sem_stage_get_tune(gm))):
        if layout:
            api.sem_stage_set_layout(gm, *layout)
        outs.append(torch.zeros_like(q))
        api.sem_stage(gm, 0.75, 0.25, 0.01, q, q, outs[-1], api.SEM_FP64)
    torch.cuda.synchronize()
    assert torch.equal(*outs) != owner
    for x, y in zip(*(o.view(5, -1) for o in outs)):
        assert float((x - y).norm()) <= TOL64 * float(y.norm())
    assert float(outs[1].abs().max()) > 0


@pytest.mark.parametrize("nx,owner", [(160, True), (164, False)])
def test_state_bytes(nx, owner):
    """2.10e9 and 2.15e9 bytes of state, rows of 511 levels."""
    _against_named(2, nx, 160, 255, owner)


@pytest.mark.parametrize("N,nx,ny,nz,owner", [
    (6, 20, 32, 1, True), (6, 21, 31, 1, False), (7, 16, 24, 2, True), (7, 17, 23, 2, False), (7, 16, 32, 8, True),
    (7, 19, 27, 8, False), (7, 6, 6, 1, False), (8, 16, 32, 1, True), (8, 19, 27, 1, False), (8, 34, 34, 1, True)])
def test_side_columns(N, nx, ny, nz, owner):
    _against_named(N, nx, ny, nz, owner, periodic=False)


@pytest.mark.parametrize("N,owner", [(7, True), (8, True)])
def test_side_columns_of_levels(N, owner):
    """175 columns of two levels, a third of them beside the other level."""
    fine = [(i, j) for i in range(3, 8) for j in range(3, 8)]
    cols = [(0, i, j) for i in range(10) for j in range(10) if (i, j) not in fine]
    cols += [(1, 2 * i + a, 2 * j + b) for i, j in fine for a in (0, 1) for b in (0, 1)]
    _against_named(N, 10, 10, 1, owner, columns=np.array(cols))


@pytest.mark.parametrize("nx,ny,nz,owner", [(24, 32, 2, True), (10, 77, 2, False), (16, 32, 1, True), (19, 27, 1, False)])
def test_columns_at_n7(nx, ny, nz, owner):
    _against_named(7, nx, ny, nz, owner)
