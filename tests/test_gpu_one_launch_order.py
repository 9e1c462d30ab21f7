"""Standard CG on meshes whose cells are in no order: a solve in one launch must
not gather past the L2 caches there (a line of 64 B for every slot; twice the
launches' time), and gives the launches' bits in either order."""
import time

import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say
from tests.test_gpu_resident import STAR, fv, stencil  # noqa: F401

pytestmark = pytest.mark.gpu


def shuffled(case, seed=1):
    """The case with its cells in random order."""
    p = np.random.default_rng(seed).permutation(case.n)
    o, n = p[case.owner], p[case.neighbour]
    lo, hi = np.minimum(o, n), np.maximum(o, n)
    k = np.lexsort((hi, lo))
    back = np.argsort(p)
    return fc.Case("shuffled", (case.n, 1, 1), case.n, lo[k].astype(np.int32), hi[k].astype(np.int32), case.diag[back],
                   case.upper[k], case.upper[k].copy(), case.b[back])


CASES = {
    "cube": lambda: fc.varcoef((91, 91, 91), seed=2, permute=False),
    "star": lambda: stencil(700, 700, STAR, 7),
    "small cube": lambda: fc.varcoef((50, 50, 50), seed=2, permute=False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_cg_on_shuffled_cells(fv, monkeypatch, name):  # noqa: F811
    import torch

    dc = DevCase(shuffled(CASES[name]()))
    for method in ("cg", "pipecg"):
        best, got = {}, {}
        for on in ("0", "1"):
            say("shuffled", name, method, on)
            monkeypatch.setenv("FVPCG_RESIDENT", on)
            times = []
            for _ in range(6):
                x = torch.zeros_like(dc.b)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                got[on], st = fv.solve(dc.A, dc.b, x=x, tol=0.0, maxit=60, method=method)
                times.append(time.perf_counter() - t0)
            assert st["one_launch"] == int(on)
            best[on] = min(times)
        assert torch.equal(got["0"], got["1"])
        say("shuffled", name, method, "one launch / launches:", round(best["1"] / best["0"], 2))
        assert best["1"] <= 1.25 * best["0"]  # 1.0 and less; 1.6 (star) and 1.9 past the caches
    dc.close()
