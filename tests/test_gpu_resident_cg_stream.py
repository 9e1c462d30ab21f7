"""Standard CG of 0.5M to 4.2M cells, all iterations in one launch, against the
launch-per-iteration path: 8 and 16 tiles of 1,024 rows per member, full and ragged,
the first size past them (launches on both sides), rows of 4, 6 and 8 slots,
int16 and int32 columns, both preconditioners, a warm start, a solve to a
tolerance, and a team that may not meet.  Both form every sum from the same
expressions in the same order, so they agree bit for bit."""
import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say, to_dev
from tests.test_gpu_resident import LINE, STAR, fv, solve, stencil  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = {
    "cube-830k-int32": (lambda: fc.varcoef((94, 94, 94), seed=12, permute=False), "0"),
    "star-600k": (lambda: stencil(800, 750, STAR, 13), "1"),
    "line-1.05M": (lambda: stencil(1050001, 1, LINE, 14), "1"),
    "cube-2097152": (lambda: fc.varcoef((128, 128, 128), seed=15, permute=False), "1"),
    "cube-2.1M": (lambda: fc.varcoef((129, 128, 128), seed=16, permute=False), "1"),
    "cube-3.4M-int32": (lambda: fc.varcoef((150, 151, 152), seed=17, permute=False), "0"),
    "cube-4194304": (lambda: fc.varcoef((128, 128, 256), seed=18, permute=False), "1"),
    "cube-4.2M": (lambda: fc.varcoef((161, 162, 162), seed=17, permute=False), "1"),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_streamed_cg_equals_launches(fv, monkeypatch, name):  # noqa: F811
    import torch

    make, col16 = SHAPES[name]
    monkeypatch.setenv("FVPCG_COL16", col16)
    case = make()
    dc = DevCase(case)
    x0 = to_dev(np.random.default_rng(1).uniform(-1, 1, case.n))
    for kw in (dict(tol=0.0, maxit=8), dict(tol=0.0, maxit=7, x0=x0, precond="none"), dict(tol=3e-2, maxit=400)):
        got = []
        for mode in ("launches", "one launch", "no-time"):
            say("streamed cg", name, mode, kw.get("tol"), kw["maxit"])
            monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0" if mode == "no-time" else "20")
            got.append(solve(fv, monkeypatch, dc, mode != "launches", method="cg", **kw))
        (xa, sa) = got[0]
        for xb, sb in got[1:]:
            for k in ("iters", "status", "b_norm", "r0_norm", "rel_res", "true_rel_res"):
                assert sa[k] == sb[k], k
            assert torch.equal(xa, xb)
    dc.close()
