"""The setup's hash products against the heap merge: the same sums in the
same order, so the hierarchies are equal bit for bit.  Meshes chosen for the
tables' edges: rows of 4 to 8 slots, a single level-1 aggregate, coarse rows
that fill the 128- and 512-slot tables and are retried in the next size, and
(theta large) rows of more columns than lanes; after a refresh too."""
import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say, to_dev
from tests.test_gpu_resident import CROSS, LINE, STAR, stencil

pytestmark = pytest.mark.gpu

CASES = {
    "line": (lambda: stencil(3000, 1, LINE, 1), 0.02),
    "cross": (lambda: stencil(90, 70, CROSS, 2), 0.0),
    "star": (lambda: stencil(80, 61, STAR, 3), 0.02),
    "tiny": (lambda: fc.varcoef((5, 5, 5), seed=4), 0.0),
    "cube": (lambda: fc.varcoef((41, 37, 33), seed=5), 0.02),
    "cube-dense": (lambda: fc.varcoef((30, 28, 26), seed=6), 0.12),
    "cavity": (lambda: fc.cavity((40, 40, 20)), 0.08),
    "unit": (lambda: fc.laplace((48, 40, 32)), 0.0),
}


@pytest.fixture(scope="module")
def fv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1505_07630_amd as fv

    fv.lib()
    return fv


def hierarchy(M):
    out = [M.levels]
    for l in range(M.levels):
        out += [M.level_info(l)["n"], M.level_info(l)["nnz"]]
        for which in ("A", "P", "R"):
            if (which == "A" and l == 0) or (which != "A" and l + 1 == M.levels):
                continue
            out += list(M.export(l, which)[:3])
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_hash_products_equal_merge(fv, monkeypatch, name):
    make, theta = CASES[name]
    case = make()
    got = {}
    for mode in ("merge", "hash"):
        say("amg products", name, mode)
        monkeypatch.setenv("FVPCG_AMG_PRODUCT", mode)
        dc = DevCase(case)
        M = fv.AMG(dc.A, theta=theta, coarse_size=8)
        first = hierarchy(M)
        rng = np.random.default_rng(7)
        scale = to_dev(rng.uniform(0.9, 1.1, case.F))
        dc.A.update(dc.diag * 1.5, dc.upper * scale)
        M.refresh()
        got[mode] = first + hierarchy(M)
        M.close()
        dc.close()
    assert len(got["merge"]) == len(got["hash"])
    for a, b in zip(got["merge"], got["hash"]):
        assert np.array_equal(a, b)
