"""The library's kept device blocks: given back when the last handle goes,
never handed out while earlier work still uses them."""
import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1505_07630_amd as fv

    fv.lib()
    return fv


def test_blocks_given_back(fv):
    import gc

    import torch

    say("memory given back")
    case = fc.varcoef((60, 50, 40), seed=3, permute=False)
    gc.collect()
    torch.cuda.synchronize()
    used = []
    for _ in range(3):
        dc = DevCase(case)
        M = fv.AMG(dc.A)
        fv.solve_amg(M, dc.b, tol=1e-8)
        fv.solve(dc.A, dc.b, method="cg", tol=1e-6)
        M.close()
        dc.close()
        del dc, M
        gc.collect()
        torch.cuda.empty_cache()
        torch.cuda.synchronize()
        used.append(torch.cuda.mem_get_info()[0])
    # the library holds nothing between the rounds: later rounds find the same free memory
    assert min(used[1:]) >= used[0] - (2 << 20), used


def test_freed_block_waits_for_its_work(fv):
    """A product still running on another stream when its matrix is freed
    keeps its values, although the next matrix takes blocks of that size."""
    import torch

    say("freed block in use")
    case = fc.varcoef((100, 90, 80), seed=4, permute=False)
    keep = DevCase(case)
    want = fv.spmv(keep.A, keep.b).clone()
    torch.cuda.synchronize()
    for _ in range(3):
        dc = DevCase(case)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        ys = [torch.empty_like(want) for _ in range(40)]
        with torch.cuda.stream(s):
            for y in ys:
                fv.spmv(dc.A, keep.b, y)
        dc.A.close()
        other = fv.Matrix(keep.mesh, 2.0 * keep.diag, 2.0 * keep.upper)
        torch.cuda.synchronize()
        assert all(torch.equal(y, want) for y in ys)
        other.close()
        dc.close()
    keep.close()
