"""BiCGSTAB's iterations in one launch against the launch-per-iteration path:
one workgroup, teams with one ragged tile each, teams of 256 with 2 to 16
tiles per member, the first size past them (launches on both sides), int16
and int32 columns, rows of 4 slots, 1 to 4 components of which some stop
earlier than others, both preconditioners, and a team that may not meet.

Both form every sum from the same expressions in the same order, so they
agree bit for bit."""
import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1505_07630_amd as fv

    fv.lib()
    return fv


def both(fv, monkeypatch, shape, nr, permute, precond, tol=1e-10, maxit=500, **env):
    import torch

    case = fc.momentum(shape, permute=permute)
    dc = DevCase(case, symmetric=False)
    g = np.random.default_rng(7)
    rhs = np.stack([case.b, g.standard_normal(case.n), np.zeros(case.n), case.b * 1e-3][:nr])
    if nr == 3:
        rhs[2] = g.uniform(0, 1, case.n)
    b = to_dev(rhs)
    out = []
    for on in ("0", "1"):
        monkeypatch.setenv("FVPCG_RESIDENT", on)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        out.append(fv.solve_bicgstab_multi(dc.A, b, x=torch.zeros_like(b), tol=tol, maxit=maxit, precond=precond))
    dc.close()
    (x0, s0), (x1, s1) = out
    assert torch.equal(x0, x1)
    for a, c in zip(s0, s1):
        for key in ("iters", "status", "b_norm", "r0_norm", "rel_res", "true_rel_res"):
            assert a[key] == c[key], key
    return s1


SHAPES = {
    "row": (1, 1, 1),
    "tile": (8, 8, 8),
    "ragged-teams": (17, 13, 11),
    "int32": (200, 200, 2),
    "plane-4-slots": (70, 50, 1),
    "256-teams": (32, 64, 64),
    "2-tiles": (53, 51, 60),
    "9-tiles": (103, 101, 100),
    "16-tiles": (128, 128, 128),
    "past": (128, 128, 129),
}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("nr", [1, 2, 3, 4])
def test_bicgstab_resident_equals_launches(fv, monkeypatch, name, nr):
    say("resident bicgstab", name, nr)
    shape = SHAPES[name]
    small = int(np.prod(shape)) < 50000
    both(fv, monkeypatch, shape, nr, permute=small and name != "int32", precond="jacobi" if nr != 2 else "none",
         maxit=500 if small else 6)


def test_bicgstab_team_that_may_not_meet(fv, monkeypatch):
    say("resident bicgstab, no time to meet")
    both(fv, monkeypatch, (30, 20, 18), 3, True, "jacobi", FVPCG_RESIDENT_MEET_MS="0")
