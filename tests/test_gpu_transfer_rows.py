"""The transfer kernel against the oracle's element-wise transfer, at row
lengths that end inside, at the end of and just past a 128-byte line, with
arrays aligned to 16 bytes and to 8 only: the padding of the input is never
read into the result, that of the output is zero, and the alignment changes no
bit.  The layouts split and merge columns, so that rows of one, a few and (at
the higher orders) hundreds of nodes occur."""

import numpy as np
import pytest

from harness import match, oracle_mesh
from oracle import adapt
from test_gpu_adapt import case_with, family_flags, random_layout, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nz", [(1, 1), (3, 5), (4, 4), (5, 3), (7, 9), (8, 2)])
def test_transfer_rows_match_oracle(N, nz):
    import torch
    from paper_2410_21607_amd import api
    say("transfer rows", N, nz)
    rng = np.random.default_rng(N)
    z = np.linspace(0.0, 20e3, nz + 1)
    a_cols = random_layout(3, 4, 4, 2, True)
    ca = case_with(a_cols, N, True)
    ca["z_edges"] = z
    ga = api.Mesh.from_case(ca)
    b_cols = api.sem_adapt_columns(ga, a_cols, family_flags(a_cols, rng), 3)
    cb = case_with(b_cols, N, True)
    cb["z_edges"] = z
    gb = ga.with_columns(b_cols)
    oa, ob = oracle_mesh(ca), oracle_mesh(cb)
    pa, pb = match(oa.node_xyz, ga.node_xyz(), ca), match(ob.node_xyz, gb.node_xyz(), cb)
    q = rng.standard_normal((5, oa.n_dof))
    want = adapt.transfer(oa, ob, q)
    flat = ga.unpack(q[:, pa])
    nzn = ga.info["nzn"]
    flat.view(5, -1, ga.ldz)[:, :, nzn:] = float("nan")
    T = api.Transfer(ga, gb)
    outs = []
    for shift_in, shift_out in [(0, 0), (1, 0), (0, 1), (1, 1)]:
        src = torch.empty(ga.n_state + 1, dtype=torch.float64, device="cuda")[shift_in:][:ga.n_state]
        src.copy_(flat)
        out = torch.full((gb.n_state + 1,), float("nan"), dtype=torch.float64, device="cuda")[shift_out:][:gb.n_state]
        api.sem_transfer_apply(T, src, out)
        torch.cuda.synchronize()
        assert torch.all(out.view(5, -1, gb.ldz)[:, :, nzn:] == 0)
        got = np.empty((5, ob.n_dof))
        got[:, pb] = gb.pack(out)
        assert np.max(np.abs(got - want)) <= 1e-13 * np.max(np.abs(want))
        outs.append(out.clone())
    assert all(torch.equal(outs[0], o) for o in outs[1:])
