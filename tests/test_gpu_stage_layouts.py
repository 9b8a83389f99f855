"""Which launches a layout stands for: a named thread order or chunk runs the
coloured launches (the default layout the owner kernel, which sums in another
order), the reported layout restores them, and the autotuner measures both."""

import numpy as np
import pytest

from oracle import metrics
from synth import cases, columns
from test_gpu_parity import TOL64, say

pytestmark = pytest.mark.gpu


class Setup:
    def __init__(self, name, kw):
        import torch
        from paper_2410_21607_amd import api
        self.torch, self.api = torch, api
        self.c = c = cases.get(name, **kw)
        self.gm = api.Mesh.from_case(c)
        bg = cases.reference_state(c, self.gm.coords()[2])
        self.gm.set_reference(bg["rho0"], bg["theta0"], bg["dtheta0dz"])
        self.q_g = self.gm.unpack(cases.initial_state(c, self.gm.node_xyz()))


def _kw(N, nx, ny, nz):
    return dict(N=N, nx0=nx, ny0=ny, Lx=4e5, Ly=3.5e5, columns=columns.uniform(nx, ny),
                z_edges=20e3 * np.linspace(0.0, 1.0, nz + 1) ** 1.05)


def _stage(S):
    out = S.torch.full_like(S.q_g, float("nan"))
    S.api.sem_stage(S.gm, 0.75, 0.25, 0.25 * S.c["dt"], S.q_g, S.q_g, out, S.api.SEM_FP64)
    S.torch.cuda.synchronize()
    return S.gm.pack(out)


@pytest.mark.parametrize("N,named", [(2, (0, 4)), (4, (0, 4)), (4, (2, 4)), (4, (3, 2)), (4, (2, 0)), (7, (0, 1))])
def test_named_layout_runs_the_coloured_launches(N, named):
    say("named layout", N, named)
    S = Setup("small_uniform", _kw(N, 4, 4, 5))
    api = S.api
    default = _stage(S)
    assert api.sem_stage_get_layout(S.gm) == (0, 0)
    api.sem_stage_set_layout(S.gm, *named)
    coloured, back = _stage(S), api.sem_stage_get_layout(S.gm)
    assert back[0] == named[0] and back[1] > 0
    assert not np.array_equal(coloured, default)
    assert metrics.rel_l2(coloured, default, metrics.STATE_FLOORS).max() <= TOL64
    for layout, want in [((0, 0), default), (back, coloured), ((0, 0), default)]:
        api.sem_stage_set_layout(S.gm, *layout)
        assert np.array_equal(_stage(S), want)
    api.sem_stage_tune(S.gm, 1)
    tuned = _stage(S)
    api.sem_stage_set_layout(S.gm, 0, 1)
    assert np.array_equal(_stage(S), tuned) and not np.array_equal(tuned, default)


def _tuned(S, prec):
    api = S.api
    lpc, ms = api.sem_stage_autotune(S.gm, S.q_g, S.q_g.clone(), S.torch.zeros_like(S.q_g), prec, reps=5)
    say("  tuned", prec, lpc, ms, api.sem_stage_get_layout(S.gm))
    assert lpc == api.sem_stage_get_tune(S.gm)
    return api.sem_stage_get_layout(S.gm)


def test_autotuner_measures_the_coloured_launches():
    """Two layers on 100 x 100 columns leave the owner kernel's chunk of eight at
    N = 3 mostly empty: it takes twice the time of the coloured launches.  On 16
    x 16 columns of 20 layers at N = 7 it takes a third."""
    say("autotuner")
    S = Setup("small_uniform", _kw(3, 100, 100, 2))
    assert _tuned(S, S.api.SEM_FP64) != (0, 0)
    S = Setup("small_uniform", _kw(7, 16, 16, 20))
    default = _stage(S)
    assert _tuned(S, S.api.SEM_FP64) == (0, 0)
    assert np.array_equal(_stage(S), default)
    # tuned for float, a double stage keeps the owner kernel
    _tuned(S, S.api.SEM_FP32)
    assert np.array_equal(_stage(S), default)
