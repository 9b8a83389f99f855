"""The element passes of the refinement side (flags, features, maximum wind) at
the sizes where their chunks of layers can go wrong: layer counts below, at and
just past a workgroup's layers for every order, hanging columns, both criteria,
rows of odd and even length; against the oracle, with the tolerance of the
feature test (float32 outputs) and exact flags (thresholds in gaps between
element maxima)."""

import numpy as np
import pytest

from harness import match, oracle_mesh
from oracle import amr, assembly, forecast
from synth import cases
from test_gpu_forecast import SCALE, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nz,criterion", [
    (1, 1, 1), (1, 17, 0), (2, 9, 1), (3, 8, 0), (3, 10, 1), (4, 4, 1), (4, 5, 0), (4, 9, 1), (5, 3, 1), (5, 7, 0),
    (6, 2, 1), (6, 3, 0), (7, 2, 1), (8, 2, 0)])
def test_element_passes_match_oracle(N, nz, criterion):
    import torch
    from paper_2410_21607_amd import api
    say("element passes", N, nz, criterion)
    c = cases.get("small_amr3", N=N)
    c["z_edges"] = np.linspace(0.0, 20e3, nz + 1)
    gm = api.Mesh.from_case(c)
    hxy, _, z = gm.coords()
    bg = cases.reference_state(c, z)
    gm.set_reference(bg["rho0"], bg["theta0"], bg["dtheta0dz"])
    om = oracle_mesh(c)
    perm = match(om.node_xyz, gm.node_xyz(), c)
    q = cases.initial_state(c, om.node_xyz)
    rng = np.random.default_rng(N)
    q[1:3] += 0.5 * rng.standard_normal(q[1:3].shape)
    qp = q * (1.0 + 0.05 * rng.standard_normal(q.shape))
    ne, nc = gm.info["n_elem"], gm.info["n_col"]
    ref = cases.reference_state(c, om.zl)
    qL, qLp = assembly.scatter(om, q), assembly.scatter(om, qp)
    crit = amr.criterion_speed(qL) if criterion == 0 else amr.criterion_vorticity(om, qL)
    cmax = crit.reshape(ne, -1).max(1)
    srt = np.unique(cmax)
    thr = np.sort(0.5 * (srt + np.roll(srt, -1))[np.argsort(np.diff(srt))[::-1][:2]])
    plain = rng.integers(-1, 2, size=ne).astype(np.int8)
    want, dem_o = forecast.features(om, qL, qLp, plain, dict(rho0=ref["rho0"], theta0=ref["theta0"]), c["phys"],
                                    criterion, thr, 2, SCALE)
    dq, dqp = gm.unpack(q[:, perm]), gm.unpack(qp[:, perm])
    feat = torch.zeros(ne * 16, dtype=torch.float32, device="cuda")
    i8 = lambda n: torch.full((n,), 9, dtype=torch.int8, device="cuda")
    dem, ae, ac = i8(ne), i8(ne), i8(nc)
    api.amr_features(gm, dq, dqp, torch.as_tensor(plain).cuda(), criterion, thr, 2, SCALE, feat, dem)
    api.amr_flag(gm, dq, criterion, thr, 2, ae, ac)
    got = feat.cpu().numpy().reshape(ne, 16).astype(np.float64)
    assert np.all(np.abs(got - want) <= 2e-6 * np.abs(want) + 1e-6)
    np.testing.assert_array_equal(dem.cpu().numpy(), dem_o)
    lv = np.repeat(np.asarray(c["columns"])[:, 0], nz)
    flags = np.where((lv < 2) & (cmax > thr[np.minimum(lv, 1)]), 1, np.where((lv > 0) & (cmax <= thr[lv - 1]), -1, 0))
    np.testing.assert_array_equal(ae.cpu().numpy(), flags)
    # maximum wind over a box: the root of the largest square, one rounding
    # of each product and sum and of the root
    wind = torch.zeros(1, dtype=torch.float64, device="cuda")
    box = (-1.2e5, 0.8e5, -1e5, 1.5e5)
    api.sem_max_wind(gm, dq, box, wind)
    inside = (hxy[:, 0] >= box[0]) & (hxy[:, 0] <= box[1]) & (hxy[:, 1] >= box[2]) & (hxy[:, 1] <= box[3])
    u = gm.pack(dq).reshape(5, len(hxy), -1)[1:3, inside]
    assert abs(float(wind.item()) - np.hypot(u[0], u[1]).max()) <= 4e-16 * float(wind.item())
