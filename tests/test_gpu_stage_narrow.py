"""Stages on meshes where a column, or a 2 x 2 block of columns, is its own
neighbour across a periodic side (one column wide, two columns wide): two of
its positions are one node.  Every path that updates nodes in place (float,
first order, dissipation, terrain, the block layout) against the oracle, at
the bars of the same paths on other meshes (FP64 1e-12, float 1e-6, floor-scaled
relative L2 per field)."""

import numpy as np
import pytest

from oracle import assembly, metrics, timestep
from synth import columns
from test_gpu_parity import TOL64, Setup, say
from test_gpu_terrain import Setup as TerrainSetup

pytestmark = pytest.mark.gpu

# one wide with the second column refined: its four children wrap as a block
REFINED = np.array([(0, 0, 0)] + [(1, a, 2 + b) for b in (0, 1) for a in (0, 1)] + [(0, 0, 2), (0, 0, 3)])
MESHES = {
    "one_wide": dict(nx0=1, ny0=3, columns=columns.uniform(1, 3)),
    "one_column": dict(nx0=1, ny0=1, columns=columns.uniform(1, 1)),
    "one_wide_walls": dict(nx0=3, ny0=1, columns=columns.uniform(3, 1), periodic_x=False),
    "one_wide_refined": dict(nx0=1, ny0=4, columns=REFINED),
    "two_wide": dict(nx0=2, ny0=4, columns=columns.uniform(2, 4)),
    "two_by_two": dict(nx0=2, ny0=2, columns=columns.uniform(2, 2)),
}
LAYOUTS = [(0, 0), (0, 1), (2, 2), (1, 0), (1, 2)]


def _kw(N, mesh):
    return dict(N=N, Lx=4e5, Ly=3.5e5, z_edges=20e3 * np.linspace(0.0, 1.0, 6) ** 1.05, **MESHES[mesh])


def _stage(S, q, qn, co, prec):
    out = S.torch.full_like(q, float("nan"))
    S.api.sem_stage(S.gm, *co, qn, q, out, prec)
    S.torch.cuda.synchronize()
    return S.to_oracle_order(out)


@pytest.mark.parametrize("mesh", MESHES)
@pytest.mark.parametrize("kind", ["order1", "float", "dissipation", "plain"])
def test_narrow_box_stage(mesh, kind):
    say("narrow", mesh, kind)
    S = Setup("small_uniform", _kw(1 if kind == "order1" else 4, mesh))
    phys = dict(S.c["phys"])
    if kind == "dissipation":
        phys.update(Cs=0.21, sponge_gamma=0.05, sponge_depth=8000.0)
        S.gm.set_dissipation(0.21, 0.05, 8000.0)
    co = timestep.stage_coefficients(1, S.c["dt"])
    qn_or = S.q_or * 1.01
    qn = S.gm.unpack(qn_or[:, S.perm])
    want = timestep.stage_update(*co, qn_or, S.q_or, assembly.rhs(S.om, S.q_or, S.ref, phys))
    prec, tol = (S.api.SEM_FP32, 1e-6) if kind == "float" else (S.api.SEM_FP64, TOL64)
    for layout in LAYOUTS:
        if layout[0] == 1 and (kind == "order1" or mesh in ("one_wide", "one_column", "one_wide_walls")):
            continue                               # no blocks
        S.api.sem_stage_set_layout(S.gm, *layout)
        err = metrics.rel_l2(_stage(S, S.q_g, qn, co, prec), want, metrics.STATE_FLOORS)
        say("  layout", layout, "rel", err)
        assert err.max() <= tol, layout


@pytest.mark.parametrize("mesh", [m for m in MESHES if m != "one_wide_walls"])
def test_narrow_terrain_stage(mesh):
    say("narrow terrain", mesh)
    S = TerrainSetup("small_uniform", _kw(4, mesh), "hills")
    want = S.oracle_rhs(S.q_or)
    for layout in [(0, 0), (2, 2)]:
        S.api.sem_stage_set_layout(S.gm, *layout)
        err = metrics.rel_l2(S.gpu_rhs(), want, metrics.RHS_FLOORS)
        say("  layout", layout, "rel", err)
        assert err.max() <= TOL64, layout
